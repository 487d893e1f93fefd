// 2D extension of the EV-FDLB step for MI355X (gfx950): a fluid homogeneous
// in z, F(x, y, p_x, p_y) = int f dp_z and G = int p_z^2/2 f dp_z on the
// tensor-product Gauss-Hermite set (p_k, p_l), k, l < 16.  The paper solves
// the 1D model and names more dimensions as the next goal (conclusions); the
// same ingredients reduced over p_z give the right-hand side
//   L = -p . grad f - F . grad_p f - nu (f - f^S) + J1
// with the Shakhov f^S (Sec. II B) and J1 (eq:J1) reduced over p_z, the
// mean-field force of eq:force integrated along z, and the averaged density
// of Sec. II A integrated along z.
//
// State d_f[2][ny][nx][16][16]: node-major, the 256 velocities of a node
// contiguous.  One TVD-RK3 stage is two kernels:
//   fields_kernel  32 x 16 (small grids: 16 x 8) nodes per workgroup, density
//                  tile with the force
//                  radius as halo in LDS: n, u, T, q from the raw velocity
//                  sums, disc-averaged density, contact value (eq:carnstar),
//                  force (antisymmetric cell pairs), transport
//                  (eq:viscosity, eq:tau, eq:prandtl), 4th-order central
//                  gradients of X = n^2 chi T, T and u along x and y.
//   fused_kernel   one workgroup per strip of 8 columns, distribution and
//                  segment of rows, all 256 velocities: WENO-5 faces along y
//                  from a ring of rows in registers and along x from the row
//                  in LDS, (Dp x I) and (I x Dp) on the f64 MFMA, Hermite
//                  equilibrium, Shakhov and J1 terms, f^(s) = a f^n +
//                  b f^(s-1) + c L(f^(s-1)), and the raw velocity sums of
//                  f^(s) for the next stage's fields.
#include "evlb2d.h"

#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <new>

#include "tables.h"

namespace evlb2d {
namespace {

// Workgroups go to the eight XCDs in turn (workgroup b to XCD b mod 8), and
// each XCD has its own L2.  xcd_block gives XCD x the contiguous blocks
// x q + min(x, r) + i (nb = 8 q + r), so that neighbouring tiles, which share
// halo lines, run on one XCD.  A bijection of 0 .. nb - 1.
__device__ __forceinline__ unsigned xcd_block(unsigned b, unsigned nb) {
  const unsigned q = nb >> 3, r = nb & 7u;
  const unsigned x = b & 7u, i = b >> 3;
  return x * q + (x < r ? x : r) + i;
}

constexpr int Q = 16;
constexpr int V = Q * Q;
constexpr int HMAX = 24;  // max halo of the fields tile (force radius / averaging disc + 2)

enum {
  F_N, F_UX, F_UY, F_T, F_SQX, F_SQY, F_NU, F_PRE, F_FX, F_FY,
  F_AX, F_AY, F_BX, F_BY, F_UXX, F_UXY, F_UYX, F_UYY, NF
};

struct Dev {
  int nx, ny;
  long long ntot;
  double inv_dx;
  double b;      // 2 pi sigma^3 / 3
  double eta_c;  // pi sigma^3 / 6
  double mu0c;   // 5 / (16 sigma^2 sqrt(pi))
  double weno_eps, g_ext;
  double T_iso;  // > 0: isothermal, the temperature the next stage sees
  int force_model, term_mask;
  int navg, npair, nrow, halo;  // cells of the averaging disc, pairs and rows of the force disc
  int* status;
};

// i mod n for |i| < 2^22, inv = 1 / n: the quotient of i + 1/2 is at least
// 1 / (2 n) away from an integer, the rounding of the product far less.
__device__ __forceinline__ int wrap(int i, int n, float inv) {
  return i - n * (int)floorf(((float)i + 0.5f) * inv);
}

// Raw velocity sums of one node -> n, u, T, q (Sec. II B moments with the
// reduced G carrying the p_z energy):
//   3/2 n T = sum (|xi|^2/2 F + G),  q = sum xi (|xi|^2/2 F + G).
struct Raw {
  double n, jx, jy, pxx, pxy, pyy, rx, ry, g0, hx, hy;
};

struct Moments {
  double n, ux, uy, T, qx, qy;
};

__device__ __forceinline__ Moments finish_moments(const Raw& m, int* status, double T_iso) {
  Moments o;
  o.n = m.n;
  o.ux = m.jx / o.n;
  o.uy = m.jy / o.n;
  const double u2 = o.ux * o.ux + o.uy * o.uy;
  const double tr = m.pxx + m.pyy;
  const double T = (2.0 / 3.0) * (0.5 * tr + m.g0 - 0.5 * o.n * u2) / o.n;
  o.qx = 0.5 * (m.rx - 2.0 * (o.ux * m.pxx + o.uy * m.pxy) - o.ux * tr + 2.0 * o.n * o.ux * u2) + (m.hx - o.ux * m.g0);
  o.qy = 0.5 * (m.ry - 2.0 * (o.ux * m.pxy + o.uy * m.pyy) - o.uy * tr + 2.0 * o.n * o.uy * u2) + (m.hy - o.uy * m.g0);
  o.T = T_iso > 0.0 ? T_iso : T;
  if (!(o.n > 0.0) || !(T > 0.0) || !isfinite(o.n) || !isfinite(T) || !isfinite(o.ux) || !isfinite(o.uy) ||
      !isfinite(o.qx) || !isfinite(o.qy))
    status[0] = 1;
  return o;
}

typedef double dbl2 __attribute__((ext_vector_type(2)));
// two values of a caller's array, which need not start on 16 bytes (the loads
// and stores are 16 bytes wide all the same: they need 4-byte alignment)
typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));

// ---------------------------------------------------------------------------
// raw velocity sums of a state (first stage of a step, evlb_moments).  State
// layout: distribution d, node i, velocity (k, l) at ((d ntot + i) V + Q k + l):
// the 2 KiB of a node's distribution are contiguous.  Eight lanes a node, lane
// q the velocities l = 2 q, 2 q + 1 of every k as 16-byte loads (a wavefront's
// load covers eight whole lines): per l the moments over k, sum_k p_k^m F for
// m < 4 and sum_k p_k^m G for m < 2, which the powers of p_l then weigh, and
// three exchanges among the eight lanes.  Bound by the read of the state; one
// wavefront a node with 66 shuffles took 1.40 ms at 1024 x 1024 nodes, this
// 0.90 ms (moments 1.43 and four copies, 0.82 ms: 5.3 TB/s).
// ---------------------------------------------------------------------------
constexpr int MNODES = 32;  // nodes per workgroup of 256 threads

// sum over the eight lanes 8 i .. 8 i + 7 (every lane gets it): DPP quad_perm
// xor 1 and 2, then row_half_mirror
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
  return v + __builtin_bit_cast(double, (unsigned long long)(unsigned)lo | ((unsigned long long)(unsigned)hi << 32));
}
__device__ __forceinline__ double sum8(double v) { return dpp_add<0x141>(dpp_add<0x4e>(dpp_add<0xb1>(v))); }

// raw sums [11][MNODES] of the workgroup's nodes into LDS (nodes past the
// domain repeat the last one)
__device__ __forceinline__ void velocity_sums(const Dev& D, const double* __restrict__ f,
                                              const double* __restrict__ vel, double (*S)[MNODES]) {
  const int slot = threadIdx.x >> 3, q = threadIdx.x & 7;
  const long long node = min((long long)blockIdx.x * MNODES + slot, D.ntot - 1);
  const dbl2u* F = (const dbl2u*)(f + node * V) + q;
  const dbl2u* G = (const dbl2u*)(f + (D.ntot + node) * V) + q;
  dbl2 Fv[Q], Gv[Q];
#pragma unroll
  for (int k = 0; k < Q; ++k) Fv[k] = F[k * (Q / 2)];
#pragma unroll
  for (int k = 0; k < Q; ++k) Gv[k] = G[k * (Q / 2)];
  double a[11] = {};
  dbl2 s0 = {}, s1 = {}, s2 = {}, s3 = {}, t0 = {}, t1 = {};
#pragma unroll
  for (int k = 0; k < Q; ++k) {
    const double p = vel[k], p2 = p * p, p3 = p2 * p;
    s0 += Fv[k];
    s1 += p * Fv[k];
    s2 += p2 * Fv[k];
    s3 += p3 * Fv[k];
    t0 += Gv[k];
    t1 += p * Gv[k];
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const double p = vel[2 * q + j], p2 = p * p;
    a[0] += s0[j];
    a[1] += s1[j];
    a[2] += p * s0[j];
    a[3] += s2[j];
    a[4] += p * s1[j];
    a[5] += p2 * s0[j];
    a[6] += s3[j] + p2 * s1[j];
    a[7] += p * s2[j] + p2 * p * s0[j];
    a[8] += t0[j];
    a[9] += t1[j];
    a[10] += p * t0[j];
  }
#pragma unroll
  for (int i = 0; i < 11; ++i) {
    a[i] = sum8(a[i]);
    if (q == (i & 7)) S[i][slot] = a[i];
  }
  __syncthreads();
}

// n, u, T, q of a state (evlb_moments): T is the moment temperature
__global__ __launch_bounds__(256) void moments_kernel(Dev D, const double* __restrict__ f, double* __restrict__ n,
                                                      double* __restrict__ u, double* __restrict__ T,
                                                      double* __restrict__ q, const double* __restrict__ vel) {
  __shared__ double S[11][MNODES];
  velocity_sums(D, f, vel, S);
  const int t = threadIdx.x;
  const long long node = (long long)blockIdx.x * MNODES + t, N = D.ntot;
  if (t >= MNODES || node >= N) return;
  const Raw m{S[0][t], S[1][t], S[2][t], S[3][t], S[4][t], S[5][t], S[6][t], S[7][t], S[8][t], S[9][t], S[10][t]};
  const Moments o = finish_moments(m, D.status, 0.0);
  n[node] = o.n;
  u[node] = o.ux;
  u[N + node] = o.uy;
  T[node] = o.T;
  if (q) {
    q[node] = o.qx;
    q[N + node] = o.qy;
  }
}

// raw velocity sums [11][ntot] of a state, the input of a stage's fields
__global__ __launch_bounds__(256) void raw_sums_kernel(Dev D, const double* __restrict__ f, double* __restrict__ raw,
                                                       const double* __restrict__ vel) {
  __shared__ double S[11][MNODES];
  velocity_sums(D, f, vel, S);
  for (int i = threadIdx.x; i < 11 * MNODES; i += 256) {
    const long long node = (long long)blockIdx.x * MNODES + i % MNODES;
    if (node < D.ntot) raw[i / MNODES * D.ntot + node] = S[i / MNODES][i % MNODES];
  }
}

// Reduced Maxwellian of given fields.  A workgroup takes ENODES nodes: the
// Hermite coefficients of one velocity component at unit density, a_0 = 1,
// a_1 = u, a_{m+1} = u a_m + m (T - 1) a_{m-1}, once per (node, axis); the
// expansions e_k = sum_m meq[k][m] a_m once per (node, axis, k); then the
// products, as 16-byte stores over the nodes' contiguous 2 KiB.  Bound by the
// write of the state; with all 64 lanes of a node's wavefront forming the
// coefficients and their own expansions it took 2.07 ms at 1024 x 1024 nodes,
// this 0.80 ms (5.4 TB/s).
constexpr int ENODES = 16;

__global__ __launch_bounds__(256) void equilibrium_kernel(Dev D, const double* __restrict__ n_in,
                                                          const double* __restrict__ u_in,
                                                          const double* __restrict__ T_in, double* __restrict__ f,
                                                          const double* __restrict__ meq) {
  __shared__ double sa[Q][2 * ENODES];            // a_m of column (axis, node)
  __shared__ __align__(16) double se[2][ENODES][Q];  // n e_k(u_x), e_l(u_y)
  __shared__ double sT[ENODES];
  const int t = threadIdx.x;
  const long long N = D.ntot, i0 = (long long)blockIdx.x * ENODES;
  // meq row of this thread's expansions, fetched beside the fields
  const int k = t & 15, col = t >> 4;  // column col (x) and ENODES + col (y)
  double mrow[Q];
#pragma unroll
  for (int m = 0; m < Q; ++m) mrow[m] = meq[k * Q + m];
  const long long inode = min(i0 + col, N - 1);
  const double n = n_in[inode];
  if (t < 2 * ENODES) {
    const long long node = min(i0 + (t & (ENODES - 1)), N - 1);
    const double u = u_in[t < ENODES ? node : N + node], T = T_in[node];
    double a0 = 1.0, a1 = u;
    sa[0][t] = a0;
    sa[1][t] = a1;
#pragma unroll
    for (int m = 1; m < Q - 1; ++m) {
      const double an = u * a1 + (double)m * (T - 1.0) * a0;
      a0 = a1;
      a1 = an;
      sa[m + 1][t] = an;
    }
    if (t < ENODES) sT[t] = T;
  }
  __syncthreads();
  double ex = 0.0, ey = 0.0;
#pragma unroll
  for (int m = 0; m < Q; ++m) {
    ex += mrow[m] * sa[m][col];
    ey += mrow[m] * sa[m][ENODES + col];
  }
  se[0][col][k] = n * ex;
  se[1][col][k] = ey;
  __syncthreads();
  // thread (h, kk, lp): velocities (kk, 2 lp), (kk, 2 lp + 1) of nodes h, h + 2, ..
  const int lp = t & 7, kk = (t >> 3) & 15, h = t >> 7;
#pragma unroll
  for (int i = 0; i < ENODES; i += 2) {
    const long long node = i0 + i + h;
    if (node >= N) break;
    const double e = se[0][i + h][kk];
    const dbl2 y = *(const dbl2*)&se[1][i + h][2 * lp];
    const dbl2 E = {e * y[0], e * y[1]};
    const double g = 0.5 * sT[i + h];
    *(dbl2u*)(f + node * V + Q * kk + 2 * lp) = E;
    *(dbl2u*)(f + (N + node) * V + Q * kk + 2 * lp) = dbl2{g * E[0], g * E[1]};
  }
}

// ---------------------------------------------------------------------------
// node fields
// ---------------------------------------------------------------------------
// Tile of a workgroup: TX x TY nodes, NT threads.  The force sums give a lane
// XN nodes along x and each group of TX TY / XN lanes a share of the disc's
// rows; the averaged density takes AV threads per node.
template <int TX_, int TY_, int XN_, int NT_>
struct FieldsShape {
  static constexpr int TX = TX_, TY = TY_, XN = XN_, NT = NT_, NODES = TX * TY;
  static constexpr int GX = TX + 4, GY = TY + 4;  // tile +-2 (gradient stencil)
  static constexpr int LANES = NODES / XN;        // of a group
  static constexpr int FG = NT / LANES;           // groups
  static constexpr int AV = NT >= 2 * GX * GY ? 2 : 1;
  static_assert(TX % XN == 0 && (LANES == 64 || LANES == 32) && FG % 2 == 0, "groups fill wavefronts");
  static_assert(NT >= NODES, "a thread per node");
  // Width of the density tile's rows in LDS: the tile and its halo, made 1
  // (mod XN), so that lanes XN nodes apart in x and rows apart in y hit
  // distinct banks.
  __host__ __device__ static constexpr int px(int halo) { return (TX + 2 * halo + XN - 2) / XN * XN + 1; }
  // Its size; half the groups' partial forces take its place once it has been
  // read, XN apart by one (distinct banks).
  static constexpr int PF = NODES + LANES;
  __host__ __device__ static constexpr int tile(int halo) {
    const int a = px(halo) * (TY + 2 * halo), b = FG * PF;
    return ((a > b ? a : b) + 1) & ~1;
  }
};
constexpr int ROWPAD = 16;  // empty rows after the disc's
typedef FieldsShape<32, 16, 8, 512> FieldsWide;   // grids that fill the chip
typedef FieldsShape<16, 8, 4, 512> FieldsSmall;   // small grids: a quarter of the chain per workgroup

// u_x, u_y and T from the raw sums n, j_x, j_y, P_xx, P_yy, g0 of a node
// (3/2 n T = sum |xi|^2/2 F + G); an isothermal run sees its fixed temperature
__device__ __forceinline__ void flow_of(const double (&m)[6], double T_iso, double& ux, double& uy, double& T) {
  const double n = m[0];
  ux = m[1] / n;
  uy = m[2] / n;
  const double e = 0.5 * (m[3] + m[4]) + m[5];
  T = T_iso > 0.0 ? T_iso : (2.0 / 3.0) * (e - 0.5 * n * (ux * ux + uy * uy)) / n;
}

// Mean-field force of the lane's FXN neighbouring nodes from one row of the disc: pairs
// (di, dj), di = d0 .. d0 + cnt - 1, with the coefficients c = {cx, cy} in
// order.  rp, lp: node 0's cells (d0, dj) and (-d0, -dj).  The cells of
// neighbouring nodes overlap: per pair one new value on either side serves all
// nodes, in registers that move by one cell a pair (four pairs unrolled, so
// that nothing is moved).
template <int FXN>
__device__ __forceinline__ void force_row(const double* rp, const double* lp, const dbl2* c, int cnt,
                                          double (&ax)[FXN], double (&ay)[FXN]) {
  double r[FXN + 3], l[FXN + 3];  // cells of node 0 at pair t: t + i to the right, t + i - (FXN - 1) to the left
#pragma unroll
  for (int i = 0; i < FXN - 1; ++i) {
    r[i] = rp[i];
    l[i] = lp[FXN - 1 - i];
  }
  auto pair = [&](int q, const dbl2 k) {
#pragma unroll
    for (int j = 0; j < FXN; ++j) {
      const double d = r[q + j] - l[q + FXN - 1 - j];
      ax[j] = fma(k[0], d, ax[j]);
      ay[j] = fma(k[1], d, ay[j]);
    }
  };
  int t = 0;
  for (; t + 4 <= cnt; t += 4) {
    dbl2 k[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) k[i] = c[t + i];
#pragma unroll
    for (int i = FXN - 1; i < FXN + 3; ++i) {
      r[i] = rp[t + i];
      l[i] = lp[FXN - 1 - t - i];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) pair(q, k[q]);
#pragma unroll
    for (int i = 0; i < FXN - 1; ++i) {
      r[i] = r[i + 4];
      l[i] = l[i + 4];
    }
  }
  // the last cnt - t < 4 pairs: their cells only
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    if (t + q < cnt) {
      r[q + FXN - 1] = rp[t + q + FXN - 1];
      l[q + FXN - 1] = lp[-t - q];
      pair(q, c[t + q]);
    }
  }
}

// Bound by the force sums, 628 pairs per node at a radius of 20 cells, and on
// small grids by their chain.  With one node per lane every pair reads two
// values and three coefficients from LDS and the scalar cache one wait after
// the other; here a lane takes 8 (4) neighbouring nodes, so that a pair costs a
// quarter (half) of a value, the disc's rows are shared among 8 (16) groups and
// summed through LDS, and every phase's loads are in flight together.  Per
// launch: 1024 x 1024 nodes 249 -> 157 us, 333 x 270 66 -> 30 us, 64 x 48 51 -> 11 us.
template <class SH>
__global__ __launch_bounds__(SH::NT) void fields_kernel(Dev D, const double* __restrict__ raw, double* __restrict__ fld,
                                                     const int* __restrict__ avg_ofs,
                                                     const double* __restrict__ avg_w,
                                                     const int4* __restrict__ disc_rows,
                                                     const dbl2* __restrict__ disc_c) {
  extern __shared__ double sm[];
  constexpr int FTX = SH::TX, FTY = SH::TY, FXN = SH::XN, FNT = SH::NT, FG = SH::FG, GX = SH::GX, GY = SH::GY;
  constexpr int PF = SH::PF, LANES = SH::LANES, AV = SH::AV;
  const int H = D.halo, PX = SH::px(H), PY = FTY + 2 * H;
  double* sn = sm;             // [PY][PX] density, node (x0 - H + c, y0 - H + r)
  double* sX = sn + SH::tile(H);  // [GY][GX] node (x0 - 2 + c, y0 - 2 + r)
  double* sT = sX + GX * GY;
  double* sux = sT + GX * GY;
  double* suy = sux + GX * GY;
  double* sC = suy + GX * GY;        // [FTY][FTX] contact value
  dbl2* sP = (dbl2*)(sC + SH::NODES);      // [npair] force coefficients
  double* sA = (double*)(sP + D.npair);  // [navg] averaging weights
  int* sO = (int*)(sA + D.navg);     // [navg] and offsets
  double* sF = sn;                   // [FG / 2][2][PF] partial forces, in the tile's place
  const int tid = threadIdx.x;
  // contiguous ranges of tiles per XCD (row-major over the tile grid): the
  // density halos of neighbouring tiles meet in one L2
  const unsigned tb = xcd_block(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
  const int x0 = (int)(tb % gridDim.x) * FTX, y0 = (int)(tb / gridDim.x) * FTY;
  const long long N = D.ntot;
  // density tile, u and T on the tile +-2, stencil tables: many loads in
  // flight at a time (one by one, each would wait for the one before)
  constexpr int FLB = 9;
  const int PW = FTX + 2 * H, ntile = PW * PY;
  const float inx = 1.0f / (float)D.nx, iny = 1.0f / (float)D.ny;
  int r = tid / PW, c = tid - r * PW;
  const int dr = FNT / PW, dc = FNT - dr * PW;
  for (int b = tid; b < ntile; b += FLB * FNT) {
    double v[FLB];
    int at[FLB];
#pragma unroll
    for (int q = 0; q < FLB; ++q) {
      at[q] = b + q * FNT < ntile ? r * PX + c : -1;
      v[q] = 0.0;
      if (at[q] >= 0) v[q] = raw[(long long)wrap(y0 - H + r, D.ny, iny) * D.nx + wrap(x0 - H + c, D.nx, inx)];
      r += dr;
      c += dc;
      if (c >= PW) {
        c -= PW;
        ++r;
      }
    }
#pragma unroll
    for (int q = 0; q < FLB; ++q)
      if (at[q] >= 0) sn[at[q]] = v[q];
  }
  {
    constexpr int LG = (GX * GY + FNT - 1) / FNT;
    double m[LG][6];
#pragma unroll
    for (int q = 0; q < LG; ++q) {
      const int i = tid + q * FNT, gr = i / GX, gc = i - gr * GX;
      const long long node = (long long)wrap(y0 - 2 + gr, D.ny, iny) * D.nx + wrap(x0 - 2 + gc, D.nx, inx);
      constexpr int pl[6] = {0, 1, 2, 3, 5, 8};  // n, j_x, j_y, P_xx, P_yy, g0
#pragma unroll
      for (int k = 0; k < 6; ++k) m[q][k] = i < GX * GY ? raw[pl[k] * N + node] : 1.0;
    }
    for (int i = tid; i < D.npair; i += FNT) sP[i] = disc_c[i];
    for (int i = tid; i < D.navg; i += FNT) {
      sA[i] = avg_w[i];
      sO[i] = avg_ofs[i];
    }
#pragma unroll
    for (int q = 0; q < LG; ++q) {
      const int i = tid + q * FNT;
      if (i < GX * GY) flow_of(m[q], D.T_iso, sux[i], suy[i], sT[i]);
    }
  }
  __syncthreads();
  // averaged density over the disc, contact value, X on the tile +-2; with two
  // threads per node each takes every other cell
  for (int j = tid; j < AV * GX * GY; j += FNT) {
    const int i = j / AV, part = j - AV * i;
    const int gr = i / GX, gc = i - gr * GX;
    const int ctr = (gr - 2 + H) * PX + (gc - 2 + H);
    double s0 = 0.0, s1 = 0.0;
    int t = part;
    for (; t + 7 * AV < D.navg; t += 8 * AV) {
#pragma unroll
      for (int q = 0; q < 8; q += 2) {
        s0 += sA[t + q * AV] * sn[ctr + sO[t + q * AV]];
        s1 += sA[t + (q + 1) * AV] * sn[ctr + sO[t + (q + 1) * AV]];
      }
    }
    for (; t < D.navg; t += AV) s0 += sA[t] * sn[ctr + sO[t]];
    s0 += s1;
    if (AV == 2) s0 += __shfl_xor(s0, 1);
    if (part == 0) {
      const double eta = D.eta_c * s0;
      const double om = 1.0 - eta;
      const double chi = (2.0 - eta) / (2.0 * om * om * om);
      const double n = sn[ctr];
      if (gr >= 2 && gr < FTY + 2 && gc >= 2 && gc < FTX + 2) sC[(gr - 2) * FTX + gc - 2] = chi;
      sX[i] = n * n * chi * sT[i];
    }
  }
  const int tx = tid % FTX, ty = tid / FTX;
  const double n = tid < SH::NODES ? sn[(ty + H) * PX + (tx + H)] : 1.0;
  if (D.force_model == EVLB_FORCE_EV1) {
    const int grp = LANES == 64 ? __builtin_amdgcn_readfirstlane(tid / LANES) : tid / LANES, lane = tid % LANES;
    const int fx = lane % (FTX / FXN) * FXN, fy = lane / (FTX / FXN);
    const double* ctr = sn + (fy + H) * PX + fx + H;
    double ax[FXN] = {}, ay[FXN] = {};
    int4 q = disc_rows[grp];  // dj, d0, count, first pair (count 0 past the last row)
    for (int i = grp; i < D.nrow; i += FG) {
      const int4 qn = disc_rows[i + FG];
      force_row<FXN>(ctr + q.x * PX + q.y, ctr - q.x * PX - q.y, sP + q.w, q.z, ax, ay);
      q = qn;
    }
    __syncthreads();  // the density tile is read
    // the upper half of the groups hands its sums to the lower half, which
    // leaves its own for the nodes' threads
    double* p = sF + grp % (FG / 2) * 2 * PF + lane * (FXN + 1);
    if (grp >= FG / 2) {
#pragma unroll
      for (int j = 0; j < FXN; ++j) {
        p[j] = ax[j];
        p[PF + j] = ay[j];
      }
    }
    __syncthreads();
    if (grp < FG / 2) {
#pragma unroll
      for (int j = 0; j < FXN; ++j) {
        p[j] += ax[j];
        p[PF + j] += ay[j];
      }
    }
  }
  __syncthreads();
  const int x = x0 + tx, y = y0 + ty;
  if (tid >= SH::NODES || x >= D.nx || y >= D.ny) return;
  const long long node = (long long)y * D.nx + x;
  const int g = (ty + 2) * GX + (tx + 2);
  const double T = sT[g], ux = sux[g], uy = suy[g], chi = sC[tid];
  double Fx = D.g_ext, Fy = 0.0;
  if (D.force_model == EVLB_FORCE_EV1) {
    const double* p = sF + tid / FXN * (FXN + 1) + tid % FXN;
    double sx[2] = {}, sy[2] = {};
#pragma unroll
    for (int w = 0; w < FG / 2; ++w) {
      sx[w & 1] += p[w * 2 * PF];
      sy[w & 1] += p[w * 2 * PF + PF];
    }
    Fx += sx[0] + sx[1];
    Fy = sy[0] + sy[1];
  }
  const double c12 = D.inv_dx * (1.0 / 12.0);
  const double X = sX[g];
  const double Ax = (sX[g - 2] - 8.0 * sX[g - 1] + 8.0 * sX[g + 1] - sX[g + 2]) * c12 / X;
  const double Ay = (sX[g - 2 * GX] - 8.0 * sX[g - GX] + 8.0 * sX[g + GX] - sX[g + 2 * GX]) * c12 / X;
  const double Bx = (sT[g - 2] - 8.0 * sT[g - 1] + 8.0 * sT[g + 1] - sT[g + 2]) * c12 / T;
  const double By = (sT[g - 2 * GX] - 8.0 * sT[g - GX] + 8.0 * sT[g + GX] - sT[g + 2 * GX]) * c12 / T;
  const double Uxx = (sux[g - 2] - 8.0 * sux[g - 1] + 8.0 * sux[g + 1] - sux[g + 2]) * c12;
  const double Uxy = (suy[g - 2] - 8.0 * suy[g - 1] + 8.0 * suy[g + 1] - suy[g + 2]) * c12;
  const double Uyx = (sux[g - 2 * GX] - 8.0 * sux[g - GX] + 8.0 * sux[g + GX] - sux[g + 2 * GX]) * c12;
  const double Uyy = (suy[g - 2 * GX] - 8.0 * suy[g - GX] + 8.0 * suy[g + GX] - suy[g + 2 * GX]) * c12;
  const double bn = D.b * n;
  const double yv = bn * chi;
  const double k12 = 0.16 * (1.0 + 12.0 / M_PI);
  const double k32 = 0.36 * (1.0 + 32.0 / (9.0 * M_PI));
  const double mu = D.mu0c * sqrt(T) * (1.0 / chi + 0.8 * bn + k12 * bn * bn * chi);
  const double nu = chi * n * T * (1.0 + 0.4 * yv) / mu;
  const double Pr = (2.0 / 3.0) * (1.0 + 0.6 * yv) * (1.0 + 0.8 * yv + k12 * yv * yv) /
                    ((1.0 + 0.4 * yv) * (1.0 + 1.2 * yv + k32 * yv * yv));
  const double s = (1.0 - Pr) / (5.0 * n * T * T);
  // heat flux and the status check of this node from its raw sums
  Raw m;
  m.n = n;
  m.jx = raw[N + node];
  m.jy = raw[2 * N + node];
  m.pxx = raw[3 * N + node];
  m.pxy = raw[4 * N + node];
  m.pyy = raw[5 * N + node];
  m.rx = raw[6 * N + node];
  m.ry = raw[7 * N + node];
  m.g0 = raw[8 * N + node];
  m.hx = raw[9 * N + node];
  m.hy = raw[10 * N + node];
  const Moments o = finish_moments(m, D.status, D.T_iso);
  const double vals[NF] = {n, ux, uy, T, s * o.qx, s * o.qy, nu, -bn * chi, Fx, Fy,
                           Ax, Ay, Bx, By, Uxx, Uxy, Uyx, Uyy};
#pragma unroll
  for (int i = 0; i < NF; ++i) fld[i * N + node] = vals[i];
}

// ---------------------------------------------------------------------------
// fused stage: one workgroup of sixteen wavefronts owns a strip of 8
// columns, one distribution (F or G) and all 256 velocities, and marches
// down a segment of rows
// ---------------------------------------------------------------------------
// Thread (wavefront w, lane L): column c = L & 7 and r = L >> 3; it holds the
// two velocities (k, l) = (w, r) and (w, 15 - r), a mirror pair: p_(15-l) =
// -p_l.  This is the B operand and result layout of v_mfma_f64_4x4x4 (four
// independent 4 x 4 blocks: block L >> 2 & 3, column L & 3, row or contraction
// index L >> 4; an A operand has its row in L & 3 and its contraction index in
// L >> 4), so a row's values enter the matrix units as they lie in registers:
// block (L >> 2 & 1) + 2 (r & 1), index r >> 1.  In the node-major state a
// wavefront's 16 velocities of a node are one 128-byte line, read as two
// halves by consecutive loads.
//
// What bounds it: the instructions issued per row (four wavefronts per SIMD)
// and, beside them, the address lookups of the march's loads and stores: lanes
// of one instruction lie on 8 nodes' lines, neighbours never on one, so that an
// instruction takes some 54 lookups (the unit is busy 92% of a 1024 x 1024
// stage).  Whole lines per instruction through LDS, two values a lane, take 8;
// in the march that cost as much LDS work and registers (1024 x 1024 3.80 ->
// 4.03 ms a stage), so only the prologue loads that way, and the halo columns
// go four lanes to 32 bytes (64 x 48 37.1 -> 33.5 us a stage with its fields,
// 333 x 270 320 -> 311).  Against a version with 16 x 16 x 4 matrix instructions, right
// faces by DPP, per-lane coefficients and addresses formed every row, this one
// runs a 1024 x 1024 step (three stages and the entry sums) in 12.4 instead of
// 16.4 ms and 333 x 270 in 1.07 instead of 2.09 ms per step.
//
// Every wavefront sees one sign of p_k (k < 8: p_k < 0) and every register
// slot one sign of p_l.  Wavefronts of p_k < 0 hold the strip mirrored (lane
// column c is the strip's column 7 - c): the upwind side is then on the left
// for every wavefront, x faces are one piece of code, and each lane's face
// enters with |p_k|.
//
// The momentum derivatives use the mirror symmetry Dp[15-k][15-j] =
// -Dp[k][j]: with f+- = f_j +- f_(15-j), j < 8, e = S f+ and o = A f-, where S,
// A = (Dp[k][j] +- Dp[k][15-j]) / 2, (Dp f)_k = e + o and (Dp f)_(15-k) = o - e:
// two 8 x 8 products for one of 16 x 16, half the matrix work (and the 4 x 4
// blocks run at the rate of the 16 x 16 ones: 512 flops in 16 cycles).
//
// One barrier per row.  Iteration y is
//  pre(y)   (each wavefront on its own 16 velocities, no data of another
//           wavefront): the row to LDS with three halo columns each side;
//           WENO-5 faces along y from a ring of five rows per velocity in
//           registers; WENO-5 faces along x from the LDS row (each lane the
//           face on its left, the one on its right from the next lane
//           through LDS); (I x Dp) f in registers; the Shakhov + J1 collision
//           terms as a polynomial in xi_y; everything but the (Dp x I) f term
//           and the strip-edge face folded into acc(y).
//  barrier
//  post(y)  the work that reads other wavefronts' rows or writes what they
//           read: f^(s) of row y - 1 from acc(y - 1), the (Dp x I) f term and
//           the strip-edge face of row y - 1, its store and its moments
//           sum_l p_l^m f^(s), m < 4, over the wavefront's own velocities (a
//           4 x 16 product of the registers on the matrix units);
//           wavefront 0 the raw velocity sums of row y - 2 (the wavefronts'
//           moments times powers of p_k, again on the matrix units), 1 the
//           Hermite coefficients a_m(u, T) of row y + 4, 2 the expansions
//           e_k(u_x), e_l(u_y) of row y + 3, 3 the per-node collision
//           coefficients of row y + 4, 0 and 3 the collision polynomials per
//           (k, node) of row y + 2, 4 - 7 the strip-edge faces of row y, 8 -
//           15 (Dp x I) f of row y.
// What one wavefront writes and another reads crosses exactly one barrier,
// and every such buffer is double (quadruple for what is read two rows
// later), so that a wavefront one half-iteration ahead never overwrites what
// a slower one still reads.  The ring's next row, f^n and the halo columns of
// the next row and the node fields of row y + 5 are in flight across an
// iteration.
constexpr int SW = 8;            // columns per strip
constexpr int SNW = 16;          // wavefronts per workgroup
constexpr int SNT = 64 * SNW;    // threads per workgroup
constexpr int NRAW = 11;         // raw velocity sums per node: 8 of F, 3 of G
// A row in LDS, doubles: velocity (k, l) at k KS + l PS, columns -3 .. 10 of
// wavefront k's orientation at 0 .. 13 of it, its x faces and then (Dp x I) f
// of columns 0 .. 7 at 14 .. 21, a zero at 22, the strip-edge face at 23.
// Lanes of one LDS pass differ in the column and in r (PS = 24 = 8 mod 16) or
// in the column and in k (KS = 8 mod 32): distinct banks either way for these.
// Over all accesses of the march the counters show 945 conflict cycles per row
// and CU, an eighth of the row's time.
constexpr int PS = 24, KS = 16 * PS + 8;
constexpr int CDX = 14, CZERO = 22, CEDGE = 23;
constexpr int USLOT = Q * KS;
// per-node coefficients of the collision terms: the row polynomial
//   nu f^S + J1 = tf n e_k e_l (P0 + xi_y (P1 + xi_y (P2 + P3 xi_y)))
// with P0 = c0 + xi_x (c1 + xi_x (c2 + c3 xi_x)), P1 = d0 + xi_x (d1 + d2 xi_x),
// P2 = e0 + c3 xi_x, P3 = d2 (a rearrangement of the reduced Shakhov and J1
// terms), plus u_x and, scaled by the stage's c, tf n; then what every lane of
// the node takes: u_y, c nu, c F_x, c F_y
enum { CF_C0, CF_C1, CF_C2, CF_C3, CF_D0, CF_D1, CF_D2, CF_E0, CF_UX, CF_TFN, CF_UY, CF_NU, CF_FX, CF_FY, NCF };

struct FusedArgs {
  const double* fs;   // f^(s-1)
  const double* f0;   // f^n (not read when first)
  double* out;        // f^(s); may alias f0 (read pointwise before the write)
  const double* fld;  // node fields [NF][ntot]
  double* raw;        // raw velocity sums of f^(s) [NRAW][ntot] (want_mom)
  double a, b, c;     // f^(s) = a f^n + b f^(s-1) + c L(f^(s-1))
  double e3, e75;     // 0.3 and 0.75 weno_eps
  int first, want_mom;
  int nstrip, seglen;
};

// what the lanes of a row read of its node quantities
struct RowTab {
  double P[Q][SW][4];   // (k, node): c tf n e_k(u_x) (P0, P1, P2, P3)
  double E[SW][SW][6];  // (r, node): u_y, c nu, c F_x, c F_y and e_l(u_y) for l = r, 15 - r
};

struct FusedSmem {
  double U[2][USLOT];           // rows y, y - 1
  RowTab tab[2];
  double mred[2][SNW][48];      // per wavefront: moment m of column c at 8 m + c (48: distinct banks over k)
  double fl[4][NF][SW];         // node fields of a row
  double AH[4][Q][16];          // Hermite coefficients a_m(u, T) of a row, column (node, axis)
  double EK[4][2][Q][SW];       // unit-density expansions e_k(u_x) (axis 0), e_l(u_y) (axis 1)
  double CF[4][NCF][SW];        // collision coefficients of a row
  double eop[4][64];            // MFMA A operands meq[i][c + 4 b] at lane i + 16 c
  double pw[4][64];             // MFMA A operands p_(4 t + k)^m at lane m + 16 k (all four blocks)
  double vel[Q];
};
static_assert(sizeof(FusedSmem) <= 160 * 1024, "fused stage LDS exceeds 160 KiB");
static_assert(8 * (USLOT + PS) < 65536, "both row slots are reached by the 16-bit LDS offset");

// WENO-5 (Jiang & Shu) value at a face from the five values v0 .. v4 ordered
// from the upwind side (v2 is the node upwind of the face), written in the
// first differences e_m = v_(m+1) - v_m.  The candidates less v2 are g0 =
// (5 e1 - 2 e0) / 6, 6 g1 = e1 + 2 e2, 3 g2 = 2 e2 - e3 / 2; three quarters of
// the smoothness indicators are the quadratic forms e0 (e0 - 11/4 e1) + 5/2
// e1^2, e1 (e1 - 5/4 e2) + e2^2 and e3 (e3 - 11/4 e2) + 5/2 e2^2.  The weights
// d_r / (eps + beta_r)^2 normalised: with t_r = (3/4 (eps + beta_r))^2 and
// 10 d = (1, 6, 3) the value is v2 + (t1 t2 g0 + 6 t0 t2 g1 + 3 t0 t1 g2) /
// (t1 t2 + 6 t0 t2 + 3 t0 t1) (every common factor cancels).  The division
// goes through a hardware reciprocal (within 2^-24.4 on this part) and one
// third-order step r (1 + d + d^2), d = 1 - den r, which leaves the rounding of
// its own operations.  36 vector instructions; the form it replaces, squares
// and products expanded one by one and two Newton steps, took 42.
// e75 = 3/4 eps; e3 = 2/5 of that, as it enters under the factor 5/2.  The
// other constants come in scalar registers too: as literals the compiler puts
// them into two-operand fused multiply-adds, each behind a register copy.
struct WenoK {
  double e3, e75, m275, m125, p25;
};

__device__ __forceinline__ double weno5(double v0, double v1, double v2, double v3, double v4, const WenoK& K) {
  const double e0 = v1 - v0, e1 = v2 - v1, e2 = v3 - v2, e3 = v4 - v3;
  const double q1 = fma(e1, e1, K.e3), q2 = fma(e2, e2, K.e3);
  double t0 = fma(e0, fma(K.m275, e1, e0), K.p25 * q1);
  double t1 = fma(e1, fma(K.m125, e2, e1), fma(e2, e2, K.e75));
  double t2 = fma(e3, fma(K.m275, e2, e3), K.p25 * q2);
  t0 *= t0;
  t1 *= t1;
  t2 *= t2;
  const double u0 = t1 * t2, u1 = t0 * t2, u2 = t0 * t1;
  const double g0 = fma(5.0 / 6.0, e1, (-1.0 / 3.0) * e0);
  const double g1x6 = fma(2.0, e2, e1);
  const double g2x3 = fma(2.0, e2, -0.5 * e3);
  const double num = fma(u2, g2x3, fma(u1, g1x6, u0 * g0));
  const double den = fma(3.0, u2, fma(6.0, u1, u0));
  const double r = __builtin_amdgcn_rcp(den);
  const double d = fma(-den, r, 1.0);
  return fma(num, fma(r, fma(d, d, d), r), v2);
}

// DPP row_ror:8: lane i of every 16-lane row takes lane i ^ 8's value
__device__ __forceinline__ double row_half(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x128, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x128, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (unsigned long long)(unsigned)lo | ((unsigned long long)(unsigned)hi << 32));
}

// lanes 32 - 63 take the value of lanes 0 - 31
__device__ __forceinline__ double half_lo(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return __builtin_bit_cast(double, (unsigned long long)lo[0] | ((unsigned long long)hi[0] << 32));
}

typedef double dbl4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double mfma4(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// Dp applied along one mirror pair: g0, g1 = (Dp f)_r, (Dp f)_(15-r) from f0,
// f1 = f_r, f_(15-r), r = L >> 3.  A block holds the indices of one parity of
// r; those of the other come from the lane 8 away.  op: S, then A, each for
// rows of the block's parity against indices of the same and of the other.
__device__ __forceinline__ void mirror_dp(const double (&op)[4], double f0, double f1, double& g0, double& g1) {
  const double a = f0 + f1, b = f0 - f1;
  double x = mfma4(op[0], a, 0.0), y = mfma4(op[2], b, 0.0);
  x = mfma4(op[1], row_half(a), x);
  y = mfma4(op[3], row_half(b), y);
  g0 = y + x;
  g1 = y - x;
}

constexpr int BUF_DWORD3 = 0x00020000;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf(const double* base) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, -1, BUF_DWORD3);
}
// A buffer of 2^31 bytes: an access at BUF_DROP is out of range with any row
// offset below 2^31, so a store there is dropped.
constexpr unsigned BUF_DROP = 0x80000000u;
__device__ __forceinline__ dbl2 bload2(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
  return __builtin_bit_cast(dbl2, __builtin_amdgcn_raw_buffer_load_b128(r, vo, so, 0));
}
__device__ __forceinline__ double bload(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0));
}
typedef unsigned u32x2 __attribute__((__vector_size__(2 * sizeof(unsigned))));
__device__ __forceinline__ void bstore(double v, __amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, vo, so, 0);
}

// Hermite coefficients a_0 .. a_15 of the unit-density expansion along one
// axis at node (column c, axis): a_0 = 1, a_1 = u, a_{m+1} = u a_m +
// m (T - 1) a_{m-1}, into AH[s][m][c + 8 axis] (the B operand layout of the
// expansion MFMA).
__device__ __forceinline__ void fused_hermite(FusedSmem& S, int s, int t) {
  const int c = t & (SW - 1), axis = t >> 3;
  const double u = S.fl[s][axis == 0 ? F_UX : F_UY][c], Tm1 = S.fl[s][F_T][c] - 1.0;
  double* a = &S.AH[s][0][t];
  double a0 = 1.0, a1 = u;
  a[0] = a0;
  a[16] = a1;
#pragma unroll
  for (int m = 1; m < Q - 1; ++m) {
    const double an = fma(u, a1, (double)m * Tm1 * a0);
    a0 = a1;
    a1 = an;
    a[16 * (m + 1)] = an;
  }
}

// Per-node coefficients of the collision row polynomial of one
// distribution (d: F or G) from the node fields of column c (fl[s]) into
// CF[s].
__device__ __forceinline__ void fused_coeffs(const Dev& D, FusedSmem& S, int s, int c, int d, double cc) {
  const double* fl = &S.fl[s][0][0];
#define FL(i) fl[(i) * SW + c]
  const bool j0 = (D.term_mask & EVLB_TERM_J0) != 0;
  const bool j1 = (D.term_mask & EVLB_TERM_J1) != 0;
  const double T = FL(F_T), invT = 1.0 / T;
  const double nu = j0 ? FL(F_NU) : 0.0;
  const double pre = j1 ? FL(F_PRE) : 0.0;
  const double th0 = d == 0 ? 4.0 : 2.0;
  const double Sx = fma(nu, FL(F_SQX), 0.3 * pre * FL(F_BX));
  const double Sy = fma(nu, FL(F_SQY), 0.3 * pre * FL(F_BY));
  const double C = 0.2 * pre * (FL(F_UXX) + FL(F_UYY));
  const double W4 = 0.4 * pre * invT;
  double* cf = &S.CF[s][0][c];
  cf[CF_C0 * SW] = fma(-th0, C, nu);
  cf[CF_C1 * SW] = fma(-th0, Sx, pre * FL(F_AX));
  cf[CF_C2 * SW] = fma(invT, C, W4 * FL(F_UXX));
  cf[CF_C3 * SW] = invT * Sx;
  cf[CF_D0 * SW] = fma(-th0, Sy, pre * FL(F_AY));
  cf[CF_D1 * SW] = W4 * (FL(F_UXY) + FL(F_UYX));
  cf[CF_D2 * SW] = invT * Sy;
  cf[CF_E0 * SW] = fma(invT, C, W4 * FL(F_UYY));
  cf[CF_UX * SW] = FL(F_UX);
  cf[CF_TFN * SW] = (j0 || j1) ? cc * (d == 0 ? 1.0 : 0.5 * T) * FL(F_N) : 0.0;
  cf[CF_UY * SW] = FL(F_UY);
  cf[CF_NU * SW] = cc * nu;
  cf[CF_FX * SW] = cc * FL(F_FX);
  cf[CF_FY * SW] = cc * FL(F_FY);
#undef FL
}

// e_k = sum_m meq[k][m] a_m for the 16 columns (node, axis) of a row on the
// f64 MFMA (B element [c][col] = a_{c + 4 b}(col) from lane col + 16 c;
// result e_{4 j + c}(col) in register j of that lane), into EK[s].
__device__ __forceinline__ void fused_expansions(FusedSmem& S, int s, int L) {
  const int c4 = L >> 4, col16 = L & 15;
  dbl4 e = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int b = 0; b < 4; ++b)
    e = __builtin_amdgcn_mfma_f64_16x16x4f64(S.eop[b][L], S.AH[s][c4 + 4 * b][col16], e, 0, 0, 0);
#pragma unroll
  for (int j = 0; j < 4; ++j) S.EK[s][col16 >> 3][4 * j + c4][col16 & 7] = e[j];
}

// Row table of a row: lane (k = 8 h + (L >> 3), node c = L & 7) forms the
// polynomial of its (k, node) and copies e_l(u_y) of l = k and half of the
// per-node values.
__device__ __forceinline__ void fused_rowtab(FusedSmem& S, int s, RowTab& t, int h, int L) {
  const int k = 8 * h + (L >> 3), c = L & 7;
  const double* cf = &S.CF[s][0][c];
  const double x = S.vel[k] - cf[CF_UX * SW];
  const double c3 = cf[CF_C3 * SW], d2 = cf[CF_D2 * SW];
  const double P0 = fma(x, fma(x, fma(c3, x, cf[CF_C2 * SW]), cf[CF_C1 * SW]), cf[CF_C0 * SW]);
  const double P1 = fma(x, fma(d2, x, cf[CF_D1 * SW]), cf[CF_D0 * SW]);
  const double P2 = fma(c3, x, cf[CF_E0 * SW]);
  const double tfe = cf[CF_TFN * SW] * S.EK[s][0][k][c];
  double* p = &t.P[k][c][0];
  p[0] = tfe * P0;
  p[1] = tfe * P1;
  p[2] = tfe * P2;
  p[3] = tfe * d2;
  double* e = &t.E[h == 0 ? L >> 3 : 7 - (L >> 3)][c][0];
  e[4 + h] = S.EK[s][1][k][c];
  e[2 * h] = cf[(CF_UY + 2 * h) * SW];
  e[2 * h + 1] = cf[(CF_UY + 2 * h + 1) * SW];
}

// Raw velocity sums of row y from the wavefronts' moments M_i(k) = sum_l p_l^i
// f(k, l) in mred[s]: sum_k p_k^m M_i(k) on the matrix units, K = 16
// wavefronts; lane L receives m = L >> 4 of column L & 7 for i = L >> 3 & 1
// (first chain) and i + 2 (second).
//   F: n 00, j_x 10, j_y 01, P_xx 20, P_xy 11, P_yy 02, r_x 30 + 12, r_y 21 + 03
//   G: g0 00, h_x 10, h_y 01         (digits: m, i)
__device__ __forceinline__ void fused_raw_sum(const Dev& D, const FusedArgs& A, const FusedSmem& S, int d, int s, int L,
                                              int x0, int y) {
  const int m = L >> 4, i = (L >> 3) & 1, c = L & 7;
  const double* mr = &S.mred[s][m][L & 15];  // element (k, L & 15) of index k = 4 t + (L >> 4)
  double u = 0.0, v = 0.0;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    u = mfma4(S.pw[t][L], mr[192 * t], u);
    if (d == 0) v = mfma4(S.pw[t][L], mr[192 * t + 16], v);
  }
  const double w = half_lo(v);  // the second chain's m - 2 on the lanes of m >= 2
  if (x0 + c >= D.nx) return;
  double* raw = A.raw + (long long)y * D.nx + x0 + c;
  if (d == 0) {
    const int f = i == 0 ? (m == 0 ? 0 : (m == 1 ? 1 : (m == 2 ? 3 : 6))) : (m == 0 ? 2 : (m == 1 ? 4 : 7));
    if (m == 3 - i) u += w;
    if (i == 0 || m < 3) raw[f * D.ntot] = u;
    if (i == 0 && m == 0) raw[5 * D.ntot] = v;
  } else if (i + m < 2) {
    raw[(8 + m + 2 * i) * D.ntot] = u;
  }
}

// LDS traffic between the lanes of one wavefront, in program order
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Where the 16 velocities of wavefront w at node column c are staged, in a row
// slot: two planes apart, and two values further for the first of four columns,
// so that lanes r of four columns are on distinct banks; within columns 0 .. 21 of
// the planes, which are written again every row.
__device__ __forceinline__ int stage_line(int w, int c) { return w * KS + 2 * PS * c + 2 * (c & 3); }

template <int N>
struct RotC {
  static constexpr int value = N;
};

template <bool ADV, bool FRC, bool FIRST>
__global__ __launch_bounds__(SNT) void fused_kernel(Dev D, FusedArgs A, const double* __restrict__ velg,
                                                    const double* __restrict__ meqg,
                                                    const double* __restrict__ dpmg) {
  __shared__ __align__(16) FusedSmem S;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int L = tid & 63;
  const int nx = D.nx, ny = D.ny;
  // workgroup -> (segment, strip, distribution); contiguous ranges per XCD
  // put neighbouring strips, which share halo columns, on one L2
  const unsigned per = 2u * (unsigned)A.nstrip;
  const unsigned tb = xcd_block(blockIdx.x, gridDim.x);
  const int seg = (int)(tb / per), rr = (int)(tb - (unsigned)seg * per);
  const int strip = rr >> 1, d = rr & 1;
  const int x0 = strip * SW;
  const int ya = seg * A.seglen;
  const int yb = min(ya + A.seglen, ny);
  const double bb = FIRST ? A.a + A.b : A.b;  // the first stage has f^n = f^(s-1)
  WenoK K{A.e3, A.e75, -2.75, -1.25, 2.5};
  asm volatile("" : "+s"(K.m275), "+s"(K.m125), "+s"(K.p25));

  if (tid < 256) {
    const int b = tid >> 6;
    S.eop[b][L] = meqg[(L & 15) * Q + (L >> 4) + 4 * b];
    const double p = velg[4 * b + (L >> 4)];
    const int m = L & 3;
    S.pw[b][L] = m == 0 ? 1.0 : (m == 1 ? p : (m == 2 ? p * p : p * p * p));
  }
  if (tid < Q) S.vel[tid] = velg[tid];
  if (tid < 2 * V) S.U[tid >> 8][((tid >> 4) & 15) * KS + (tid & 15) * PS + CZERO] = 0.0;

  const long long dofs = (long long)d * V * D.ntot;
  const __amdgpu_buffer_rsrc_t rs = buf(A.fs + dofs), r0 = buf((FIRST ? A.fs : A.f0) + dofs), rf = buf(A.fld);
  auto wrapx = [&](int x) { x %= nx; return x < 0 ? x + nx : x; };
  const bool mir = w < 8;
  const int cl = L & 7, r = L >> 3;
  auto colx = [&](int c) { return mir ? x0 + SW - 1 - c : x0 + c; };  // the wavefront's orientation
  const int nc = mir ? SW - 1 - cl : cl;                                // node column of the lane
  // byte offsets of the lane's velocities (w, r), (w, 15 - r) at its column;
  // a row is rowb further; stores of columns past the domain are dropped
  const unsigned vo0 = ((unsigned)wrapx(x0 + nc) * (unsigned)V + 16u * (unsigned)w + (unsigned)r) * 8u;
  const unsigned vo1 = vo0 + (unsigned)(15 - 2 * r) * 8u;
  const unsigned vs0 = x0 + nc < nx ? vo0 : BUF_DROP, vs1 = x0 + nc < nx ? vo1 : BUF_DROP;
  // the prologue's loads: velocities (w, 2 (L & 7)) and the next of node column
  // L >> 3, whole lines
  const unsigned vol = ((unsigned)wrapx(x0 + (L >> 3)) * (unsigned)V + 16u * (unsigned)w + 2u * (unsigned)(L & 7)) * 8u;
  const unsigned rowb = (unsigned)nx * (unsigned)V * 8u;
  // the wavefront's halo, 16 velocities x 6 columns (a 128-byte line each):
  // four neighbouring lanes take 32 bytes of a line: fewer lookups than one
  // line per lane, and fewer bank conflicts at the write to LDS than 16 lanes to
  // a line (1024 x 1024 3.78 -> 3.73 ms a stage).  Lane L takes l = (L & 3) + 4
  // (L >> 4) of column -3, -2, -1, 8 for L >> 2 & 3 = 0 .. 3, and l = (L & 3) + 4
  // (L >> 3 & 3) of column 9 + (L >> 2 & 1) (lanes 32 - 63 repeat 0 - 31)
  const int hcA = (L & 12) < 12 ? ((L >> 2) & 3) - 3 : SW, hcB = SW + 1 + ((L >> 2) & 1);
  const int hlA = (L & 3) + 4 * (L >> 4), hlB = (L & 3) + 4 * ((L >> 3) & 3);
  const unsigned hvoA = ((unsigned)wrapx(colx(hcA)) * (unsigned)V + (unsigned)(16 * w + hlA)) * 8u;
  const unsigned hvoB = ((unsigned)wrapx(colx(hcB)) * (unsigned)V + (unsigned)(16 * w + hlB)) * 8u;
  // node fields [NF][ntot]: thread t < NF SW loads field t / SW of column t % SW
  const bool fthr = tid < NF * SW;
  const unsigned fvo =
      fthr ? ((unsigned)(tid / SW) * (unsigned)D.ntot + (unsigned)wrapx(x0 + (tid & (SW - 1)))) * 8u : 0u;
  const unsigned rowf = (unsigned)nx * 8u;
  const double pk = velg[w], pr = velg[r];
  // x faces, in the wavefront's orientation (uniform: in scalar registers)
  const unsigned long long cpxb = __builtin_bit_cast(unsigned long long, A.c * D.inv_dx * fabs(pk));
  const double cpx = __builtin_bit_cast(
      double, (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)cpxb) |
                  ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(cpxb >> 32)) << 32));
  const double cpy = A.c * D.inv_dx * pr;        // y faces of l = r; of l = 15 - r with the other sign
  // MFMA A operands: Dp along a mirror pair (mirror_dp), and the powers of
  // p_l of the moments, for the indices of the lane's block and their mirrors
  double dop[4], mop[2];
  {
    const int i = L & 3, par = (L >> 3) & 1, k = L >> 4;
    const double* dp = dpmg + (2 * i + par) * Q;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int j = 2 * k + (par ^ s);
      dop[s] = fma(0.5, dp[15 - j], 0.5 * dp[j]);
      dop[2 + s] = fma(-0.5, dp[15 - j], 0.5 * dp[j]);
    }
    const double p = velg[2 * k + par];
    const double p2 = p * p;
    mop[0] = i == 0 ? 1.0 : (i == 1 ? p : (i == 2 ? p2 : p * p2));
    mop[1] = (i & 1) ? -mop[0] : mop[0];
  }

  // y within 6 rows of the domain (ny >= 8)
  auto wrapy = [&](int y) { return (unsigned)(y < 0 ? y + ny : (y >= ny ? y - ny : y)); };
  auto rowso = [&](int y) { return wrapy(y) * rowb; };
  auto rowsf = [&](int y) { return wrapy(y) * rowf; };

  // ---- prologue.  The ring R5[j] holds, per velocity, five consecutive
  // rows in marching order: (y - 2 .. y + 2) for j = 1 (p_l > 0), (y - 1 ..
  // y + 3) for j = 0 (p_l < 0), so that the face between rows y and y + 1 is
  // weno5(R0 .. R4), resp. weno5(R4 .. R0), and the row dropped after the
  // face is always R0.
  double fpre[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) fpre[i] = bload(rf, fvo, rowsf(ya + i));
  dbl2 line[7];  // rows ya - 3 .. ya + 3
#pragma unroll
  for (int i = 0; i < 7; ++i) line[i] = bload2(rs, vol, rowso(ya - 3 + i));
  // f^n and the halo of row ya, node fields of row ya + 4
  double f0v[2] = {0.0, 0.0}, hv[2];
  if (!FIRST) {
    f0v[0] = bload(r0, vo0, rowso(ya));
    f0v[1] = bload(r0, vo1, rowso(ya));
  }
  hv[0] = bload(rs, hvoA, rowso(ya));
  hv[1] = bload(rs, hvoB, rowso(ya));
  double fq = bload(rf, fvo, rowsf(ya + 4));
  // node tables: fields of rows ya .. ya + 3, Hermite and collision
  // coefficients of these, expansions of ya .. ya + 2, row tables of ya, ya + 1
  if (fthr) {
#pragma unroll
    for (int i = 0; i < 4; ++i) S.fl[(ya + i) & 3][tid / SW][tid & (SW - 1)] = fpre[i];
  }
  __syncthreads();
  if (w == 1) fused_hermite(S, (ya + (L >> 4)) & 3, L & 15);
  if (w == 3 && L < 32) fused_coeffs(D, S, (ya + (L >> 3)) & 3, L & 7, d, A.c);
  __syncthreads();
  if (w < 3) fused_expansions(S, (ya + w) & 3, L);
  __syncthreads();
  if (w < 4) fused_rowtab(S, (ya + (w >> 1)) & 3, S.tab[w >> 1], w & 1, L);
  double fyl[2] = {0.0, 0.0};
  // The ring from the lines, through the wavefront's own planes of the row
  // slots, four lines at a time.
  double R5[2][5], e0, e1;
  {
    double* const ln = &S.U[0][stage_line(w, L >> 3) + 2 * (L & 7)];
    const double *const n0 = &S.U[0][stage_line(w, nc) + r], *const n1 = &S.U[0][stage_line(w, nc) + 15 - r];
    auto at = [](int a) { return a / 2 * USLOT + a % 2 * PS; };
#pragma unroll
    for (int i = 0; i < 4; ++i) *(dbl2*)(ln + at(i)) = line[i];
    wave_fence();
    e1 = n1[at(0)];
    e0 = n0[at(1)];
    R5[1][0] = n1[at(1)];
    R5[0][0] = n0[at(2)];
    R5[1][1] = n1[at(2)];
    R5[0][1] = n0[at(3)];
    R5[1][2] = n1[at(3)];
    wave_fence();
#pragma unroll
    for (int i = 4; i < 7; ++i) *(dbl2*)(ln + at(i - 4)) = line[i];
    wave_fence();
    R5[0][2] = n0[at(0)];
    R5[1][3] = n1[at(0)];
    R5[0][3] = n0[at(1)];
    R5[1][4] = n1[at(1)];
    R5[0][4] = n0[at(2)];
    wave_fence();
  }
  if (ADV) {  // the face between rows ya - 1 and ya
    fyl[0] = weno5(R5[0][3], R5[0][2], R5[0][1], R5[0][0], e0, K);
    fyl[1] = weno5(e1, R5[1][0], R5[1][1], R5[1][2], R5[1][3], K);
  }
  __syncthreads();

  double accP[2] = {0.0, 0.0}, cfxP = 0.0;  // acc and c F_x of the row before
  // Byte offsets into the shared block, formed once and held opaque, so that
  // the compiler keeps them in registers instead of deriving them again every
  // row: the lane's columns of its two planes, its halo values, its parts of
  // the row table, its moment, and two for the wavefront's own part of post:
  // (Dp x I) f at (k, 15 - k, l) or the plane of its edge face.
  char* const Sb = (char*)&S;
  unsigned b0 = 8u * (unsigned)(w * KS + r * PS + cl), b1 = 8u * (unsigned)(w * KS + (15 - r) * PS + cl);
  unsigned hA = 8u * (unsigned)(w * KS + hlA * PS + hcA + 3), hB = 8u * (unsigned)(w * KS + hlB * PS + hcB + 3);
  unsigned tP = (unsigned)(offsetof(FusedSmem, tab) + offsetof(RowTab, P)) + 32u * (unsigned)(w * SW + nc);
  unsigned tE = (unsigned)(offsetof(FusedSmem, tab) + offsetof(RowTab, E)) + 48u * (unsigned)(r * SW + nc);
  unsigned mw = (unsigned)offsetof(FusedSmem, mred) + 8u * (unsigned)(48 * w + 8 * (L >> 4) + nc);
  unsigned s0 = 0, s1 = 0;
  if (w >= 8) {
    s0 = 8u * (unsigned)(r * KS + 2 * (w - 8) * PS + 3 + SW - 1 - cl);
    s1 = 8u * (unsigned)((15 - r) * KS + 2 * (w - 8) * PS + 3 + cl);
  } else if (w >= 4) {
    s0 = 8u * (unsigned)((4 * (w - 4) + (L >> 4)) * KS + (L & 15) * PS);
  }
  asm volatile("" : "+v"(b0), "+v"(b1), "+v"(hA), "+v"(hB));
  asm volatile("" : "+v"(tP), "+v"(tE), "+v"(mw), "+v"(s0), "+v"(s1));
  auto lds = [&](unsigned o, int i) -> double& { return *((double*)(Sb + o) + i); };
  auto lds2 = [&](unsigned o, int i) -> dbl2 { return *((const dbl2*)(Sb + o) + i); };
  // One row of the march.  The ring is not shifted: row y uses the slots
  // rotated by (y - ya) mod 5 (slot (i + ROT) mod 5 holds ring entry i), and
  // row slot (y - ya) mod 2 of the shared block; the march is unrolled ten
  // rows at a time, so that every slot index is a constant and every LDS
  // address a held register plus an immediate.
  auto row = [&](auto rotc, const int y) {
    constexpr int ROT = decltype(rotc)::value;
    constexpr int p = ROT & 1;                       // slots of rows y, y - 2
    constexpr int U0 = p * USLOT, U1 = (1 - p) * USLOT;  // rows y and y - 1 in the shared block
    constexpr int TAB = p * (int)sizeof(RowTab);
    auto R = [&](int j, int i) -> double& { return R5[j][(i + ROT) % 5]; };
    double accN[2] = {0.0, 0.0}, cfxN = 0.0;
    // ---------------- pre(y) ----------------
    if (y < yb) {
      const double cur0 = R(0, 1), cur1 = R(1, 2);  // row y
      lds(b0, U0 + 3) = cur0;
      lds(b1, U0 + 3) = cur1;
      lds(hA, U0) = hv[0];
      lds(hB, U0) = hv[1];
      if (fthr) S.fl[y & 3][tid / SW][tid & (SW - 1)] = fq;  // row y + 4
      const dbl2 nA = lds2(tE + TAB, 0), nB = lds2(tE + TAB, 1);
      accN[0] = -nA[1] * cur0;
      accN[1] = -nA[1] * cur1;
      if (ADV) {
        // y faces: j = 0 upwind from above, j = 1 from below
        const double fyr0 = weno5(R(0, 4), R(0, 3), R(0, 2), R(0, 1), R(0, 0), K);
        const double fyr1 = weno5(R(1, 0), R(1, 1), R(1, 2), R(1, 3), R(1, 4), K);
        accN[0] = fma(cpy, fyl[0] - fyr0, accN[0]);
        accN[1] = fma(cpy, fyr1 - fyl[1], accN[1]);
        fyl[0] = fyr0;
        fyl[1] = fyr1;
      }
      if (FRC) {
        double gy0, gy1;
        mirror_dp(dop, cur0, cur1, gy0, gy1);
        accN[0] = fma(-nB[1], gy0, accN[0]);
        accN[1] = fma(-nB[1], gy1, accN[1]);
        cfxN = nB[0];
      }
      // collision terms
      const dbl2 PA = lds2(tP + TAB, 0), PB = lds2(tP + TAB, 1), el = lds2(tE + TAB, 2);
      const double xy0 = pr - nA[0], xy1 = -pr - nA[0];
      accN[0] = fma(el[0], fma(xy0, fma(xy0, fma(PB[1], xy0, PB[0]), PA[1]), PA[0]), accN[0]);
      accN[1] = fma(el[1], fma(xy1, fma(xy1, fma(PB[1], xy1, PB[0]), PA[1]), PA[0]), accN[1]);
      // the states behind these, so that few roundings are of the size of the result
      accN[0] = fma(bb, cur0, accN[0]);
      accN[1] = fma(bb, cur1, accN[1]);
      if (!FIRST) {
        accN[0] = fma(A.a, f0v[0], accN[0]);
        accN[1] = fma(A.a, f0v[1], accN[1]);
      }
    }
    // in flight across the rest of this iteration: node fields of row y + 5
    // (issued first: the wait for it in the next iteration then leaves the
    // later loads in flight), the ring's next row (into the slot just
    // dropped), f^n and the halo of row y + 1.  Outside the condition, and
    // past the segment too: a load under a condition would make the
    // compiler copy the register at the loop latch, which waits for every
    // load in flight.
    fq = bload(rf, fvo, rowsf(y + 5));
    R(0, 0) = bload(rs, vo0, rowso(y + 4));
    R(1, 0) = bload(rs, vo1, rowso(y + 3));
    {
      const unsigned so1 = rowso(y + 1);
      if (!FIRST) {
        f0v[0] = bload(r0, vo0, so1);
        f0v[1] = bload(r0, vo1, so1);
      }
      hv[0] = bload(rs, hvoA, so1);
      hv[1] = bload(rs, hvoB, so1);
    }
    if (ADV && y < yb) {
      // x faces from this wavefront's LDS row: each lane the face on its
      // left (in the wavefront's orientation), the face on its right from
      // the next lane (the last column reads the zero column; its right face
      // is the strip-edge face, added in post(y + 1)).  The fences keep the
      // compiler from moving a lane's reads of other lanes' values.
      asm volatile("" ::: "memory");
      const double lf0 = weno5(lds(b0, U0), lds(b0, U0 + 1), lds(b0, U0 + 2), lds(b0, U0 + 3), lds(b0, U0 + 4), K);
      const double lf1 = weno5(lds(b1, U0), lds(b1, U0 + 1), lds(b1, U0 + 2), lds(b1, U0 + 3), lds(b1, U0 + 4), K);
      lds(b0, U0 + CDX) = lf0;
      lds(b1, U0 + CDX) = lf1;
      asm volatile("" ::: "memory");
      accN[0] = fma(cpx, lf0 - lds(b0, U0 + CDX + 1), accN[0]);
      accN[1] = fma(cpx, lf1 - lds(b1, U0 + CDX + 1), accN[1]);
    }
    __syncthreads();
    // ---------------- post(y) ----------------
    {
      // f^(s) of row y - 1 (y > ya).  The stores run every iteration, into
      // an empty buffer where there is no row, so that every iteration
      // issues the same vector memory operations and the wait for a load
      // issued before them never has to drain them.
      const bool live = y > ya;
      const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(A.out + dofs), (short)0, live ? (int)0x80000000u : 0, BUF_DWORD3);
      const unsigned so = live ? rowso(y - 1) : 0u;
      double o0 = accP[0], o1 = accP[1];
      if (FRC) {
        o0 = fma(-cfxP, lds(b0, U1 + CDX), o0);
        o1 = fma(-cfxP, lds(b1, U1 + CDX), o1);
      }
      if (ADV && cl == SW - 1) {
        o0 = fma(-cpx, lds(b0, U1 + CEDGE - (SW - 1)), o0);
        o1 = fma(-cpx, lds(b1, U1 + CEDGE - (SW - 1)), o1);
      }
      bstore(o0, ro, vs0, so);
      bstore(o1, ro, vs1, so);
      if (A.want_mom) {
        // moments of this wavefront's 16 velocities per column
        const double m0 = mfma4(mop[1], o1, mfma4(mop[0], o0, 0.0));
        lds(mw, (1 - p) * (SNW * 48)) = m0 + row_half(m0);
      }
    }
    // the serial chains on the oldest wavefront of each SIMD (the arbiter
    // issues the oldest first), the strip-edge faces on the next oldest, the
    // MFMA work on the two youngest.  Their addresses come from an opaque copy
    // of the lane index, so that the compiler does not hoist them out of the
    // march and hold (or spill) them across it.
    int Lq = L;
    asm volatile("" : "+v"(Lq));
    if (w == 0) {
      if (A.want_mom && y - 2 >= ya) fused_raw_sum(D, A, S, d, p, Lq, x0, y - 2);
      if (y + 2 < yb) fused_rowtab(S, (y + 2) & 3, S.tab[p], 0, Lq);
    } else if (w == 1) {
      if (y + 4 < yb && Lq < 16) fused_hermite(S, y & 3, Lq);
    } else if (w == 2) {
      if (y + 3 < yb) fused_expansions(S, (y + 3) & 3, Lq);
    } else if (w == 3) {
      if (y + 2 < yb) fused_rowtab(S, (y + 2) & 3, S.tab[p], 1, Lq);
      if (y + 4 < yb && Lq < SW) fused_coeffs(D, S, y & 3, Lq, d, A.c);
    } else if (w >= 8) {
      if (FRC && y < yb) {
        // (Dp x I) f for l = 2 (w - 8) + lh, lane (k = r, column)
#pragma unroll
        for (int lh = 0; lh < 2; ++lh) {
          double gx0, gx1;
          mirror_dp(dop, lds(s0, U0 + lh * PS), lds(s1, U0 + lh * PS), gx0, gx1);
          lds(s0, U0 + lh * PS + CDX - 3) = gx0;
          lds(s1, U0 + lh * PS + CDX - 3) = gx1;
        }
      }
    } else if (ADV && y < yb) {
      // wavefronts 4 - 7: the strip-edge face of one velocity per lane
      lds(s0, U0 + CEDGE) = weno5(lds(s0, U0 + 8), lds(s0, U0 + 9), lds(s0, U0 + 10), lds(s0, U0 + 11),
                                  lds(s0, U0 + 12), K);
    }
    accP[0] = accN[0];
    accP[1] = accN[1];
    cfxP = cfxN;
  };
  for (int y = ya; y <= yb; y += 10) {
    row(RotC<0>(), y);
    if (y + 1 > yb) break;
    row(RotC<1>(), y + 1);
    if (y + 2 > yb) break;
    row(RotC<2>(), y + 2);
    if (y + 3 > yb) break;
    row(RotC<3>(), y + 3);
    if (y + 4 > yb) break;
    row(RotC<4>(), y + 4);
    if (y + 5 > yb) break;
    row(RotC<5>(), y + 5);
    if (y + 6 > yb) break;
    row(RotC<6>(), y + 6);
    if (y + 7 > yb) break;
    row(RotC<7>(), y + 7);
    if (y + 8 > yb) break;
    row(RotC<8>(), y + 8);
    if (y + 9 > yb) break;
    row(RotC<9>(), y + 9);
  }
  // velocity sums of the last row
  __syncthreads();
  if (A.want_mom && w == 0) fused_raw_sum(D, A, S, d, (yb - 1 - ya) & 1, L, x0, yb - 1);
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Layout {
  size_t tab_d, tab_i, f1, f2, raw, fld, status, total;
  int navg, npair, nrow, halo;
};

bool is_integer_multiple(double a, double dx, int* m) {
  const double r = a / dx;
  const long long k = llround(r);
  if (k <= 0 || std::fabs(r - (double)k) > 1e-9 * r) return false;
  *m = (int)k;
  return true;
}

Layout make_layout(const evlb_params* p, const evlb::DiscTables& t) {
  Layout L{};
  const long long N = (long long)p->nx[0] * p->ny;
  L.navg = (int)t.avg_w.size();
  L.npair = (int)t.pair_cx.size();
  L.nrow = 2 * t.pair_reach + 1;
  L.halo = t.pair_reach > t.avg_reach + 2 ? t.pair_reach : t.avg_reach + 2;
  size_t off = 0;
  L.tab_d = off;
  off += align256(sizeof(double) * (size_t)(Q + 2 * Q * Q + L.navg + (L.navg & 1) + 2 * (L.npair + 1)));
  L.tab_i = off;
  off += align256(sizeof(int) * (size_t)L.navg + sizeof(int4) * (size_t)(L.nrow + ROWPAD));
  const size_t fbytes = align256(sizeof(double) * 2 * (size_t)V * (size_t)N);
  L.f1 = off; off += fbytes;
  L.f2 = off; off += fbytes;
  off += align256(sizeof(double) * 6 * (size_t)N);  // unused: evlb_workspace_bytes stays as it was
  L.raw = off; off += align256(sizeof(double) * NRAW * (size_t)N);
  L.fld = off; off += align256(sizeof(double) * NF * (size_t)N);
  L.status = off; off += 256;
  L.total = off;
  return L;
}

// Split of the grid into workgroups of the fused stage: strips of SW columns,
// two distributions, segments of rows.  A workgroup takes a CU's whole LDS, so
// the launch runs in rounds of one workgroup per CU, and a segment costs its
// rows and about FUSED_START rows' time for its prologue: the number of
// segments that makes rounds x (rows + FUSED_START) smallest.  Measured per
// stage against about one workgroup per CU in segments of at least 16 rows:
// 64 x 48 nodes 16 segments 80, 3 segments 116 us; 333 x 270 (84 strips and
// distributions on 256 CUs) 3 segments 353, 4 segments 512 us; 600 x 400 5
// segments 896, 2 segments 1366 us; 1024 x 1024 one segment either way.  The
// start's cost from 128 x 128 to 600 x 400 nodes: 12 to 15 us, a row's 2.6 to 3.5.
constexpr int FUSED_START = 4;

void fused_shape(int nx, int ny, int cus, int* nstrip, int* nseg, int* seglen) {
  *nstrip = (nx + SW - 1) / SW;
  long long best = -1;
  for (int s = 1; s <= ny; ++s) {
    const int len = (ny + s - 1) / s;
    const int n = (ny + len - 1) / len;  // every segment non-empty
    const long long wgs = 2ll * *nstrip * n;
    const long long cost = (wgs + cus - 1) / cus * (len + FUSED_START);
    if (best < 0 || cost < best) {
      best = cost;
      *nseg = n;
      *seglen = len;
    }
  }
}

void disc_tables(const evlb_params* p, evlb::DiscTables& t) {
  evlb::build_disc_tables(p->dx, p->sigma, p->phi_sigma, p->r_cut, p->force_model == EVLB_FORCE_EV1, t);
}

template <class SH>
size_t fields_lds_bytes(int halo, int npair, int navg) {
  return sizeof(double) * ((size_t)SH::tile(halo) + 4 * (size_t)SH::GX * SH::GY + SH::NODES + 2 * (size_t)npair + navg) +
         sizeof(int) * (size_t)navg;
}

// The small tile where the wide one leaves CUs without a workgroup (64 x 48
// nodes: wide 24 us, small 11 us; 333 x 270, 187 wide tiles: 31 and 30 us).
bool fields_small(int nx, int ny, int cus) {
  typedef FieldsWide W;
  return (long long)((nx + W::TX - 1) / W::TX) * ((ny + W::TY - 1) / W::TY) < cus;
}

}  // namespace

struct Ctx {
  evlb_params p;
  int nx, ny;
  int nstrip, nseg, seglen;  // workgroups of the fused stage
  bool small;                // fields tile
  long long N;
  Layout L;
  Dev dev;
  char* ws;
  const double *vel, *meq, *dpm, *avg_w;
  const dbl2* disc_c;
  const int* avg_ofs;
  const int4* disc_rows;
  std::vector<double> hvel;
};

int validate(const evlb_params* p) {
  if (!p || p->dim != 2) return EVLB_EINVAL;
  if (p->n_sys != 1 || !p->nx) return EVLB_EINVAL;
  if (p->nx[0] < 8 || p->ny < 8) return EVLB_EINVAL;
  const long long N = (long long)p->nx[0] * p->ny;
  if (N > (1ll << 20)) return EVLB_EINVAL;  // 32-bit byte offsets within one distribution's 256 planes
  if (p->q != Q) return EVLB_EUNSUPPORTED;
  if (!(p->dx > 0) || !(p->dt > 0) || !std::isfinite(p->dx) || !std::isfinite(p->dt)) return EVLB_EINVAL;
  if (!(p->sigma > 0) || !std::isfinite(p->sigma) || !(p->phi_sigma >= 0) || !std::isfinite(p->phi_sigma))
    return EVLB_EINVAL;
  if (p->force_model < 0 || p->force_model > 2) return EVLB_EINVAL;
  if (p->force_model == EVLB_FORCE_EV2) return EVLB_EUNSUPPORTED;
  if (p->gamma != 6.0) return EVLB_EUNSUPPORTED;  // the z-integrated kernel is tabulated for gamma = 6
  if (p->term_mask & ~EVLB_TERM_ALL) return EVLB_EINVAL;
  if (!(p->weno_eps > 0) || !std::isfinite(p->g_ext)) return EVLB_EINVAL;
  if (p->exec_mode < 0 || p->exec_mode > 2) return EVLB_EINVAL;
  if (p->exec_mode == EVLB_EXEC_PERSISTENT) return EVLB_EUNSUPPORTED;
  if (p->tile_nodes != 0) return EVLB_EINVAL;
  if (p->adjoint != 0 && p->adjoint != 1) return EVLB_EINVAL;
  if (p->adjoint) return EVLB_EUNSUPPORTED;
  if (!(p->T_iso >= 0.0) || !std::isfinite(p->T_iso)) return EVLB_EINVAL;
  if ((int)std::ceil(p->sigma / p->dx) + 2 > HMAX) return EVLB_EINVAL;
  if (p->force_model == EVLB_FORCE_EV1) {
    int mf;
    if (!is_integer_multiple(p->r_cut, p->dx, &mf) || mf > HMAX) return EVLB_EINVAL;
  }
  // WENO-5 + TVD-RK3 along two axes: dt (|p_x| + |p_y|)_max / dx <= 1
  std::vector<double> v, w;
  evlb::gauss_hermite_nodes(Q, v, w);
  if (p->dt * 2.0 * v.back() / p->dx > 1.0) return EVLB_ECFL;
  return EVLB_OK;
}

size_t workspace_bytes(const evlb_params* p) {
  if (validate(p) != EVLB_OK) return 0;
  evlb::DiscTables t;
  disc_tables(p, t);
  return make_layout(p, t).total;
}

int init(const evlb_params* p, char* ws, size_t bytes, hipStream_t st, Ctx** out) {
  *out = nullptr;
  int rc = validate(p);
  if (rc) return rc;
  evlb::DiscTables t;
  disc_tables(p, t);
  const Layout L = make_layout(p, t);
  if (!ws || bytes < L.total || ((uintptr_t)ws & 255)) return EVLB_EWORKSPACE;
  Ctx* c = new (std::nothrow) Ctx();
  if (!c) return EVLB_EINVAL;
  c->p = *p;
  c->nx = p->nx[0];
  c->ny = p->ny;
  c->N = (long long)c->nx * c->ny;
  int device = -1, cus = 0;
  if (hipGetDevice(&device) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus < 1) {
    delete c;
    return EVLB_EHIP;
  }
  fused_shape(c->nx, c->ny, cus, &c->nstrip, &c->nseg, &c->seglen);
  c->small = fields_small(c->nx, c->ny, cus);
  c->L = L;
  c->ws = ws;
  evlb::TableParams tp{Q, p->dx, p->sigma, p->phi_sigma, p->gamma, p->r_cut};
  evlb::HostTables ht;
  evlb::build_tables(tp, ht);
  c->hvel = ht.vel;
  const int PX = c->small ? FieldsSmall::px(L.halo) : FieldsWide::px(L.halo);
  std::vector<double> hd;
  hd.insert(hd.end(), ht.vel.begin(), ht.vel.end());
  hd.insert(hd.end(), ht.meq.begin(), ht.meq.end());
  hd.insert(hd.end(), ht.dpm.begin(), ht.dpm.end());
  hd.insert(hd.end(), t.avg_w.begin(), t.avg_w.end());
  // the force pairs row by row of the disc (the tables list them so, di
  // ascending): rows {dj, first di, pairs, index of the first pair}
  std::vector<int4> hr;
  if (hd.size() & 1) hd.push_back(0.0);  // pairs on 16 bytes
  const size_t o_c = hd.size();
  for (int i = 0; i < L.npair; ++i) {
    if (hr.empty() || hr.back().x != t.pair_dj[i]) hr.push_back(make_int4(t.pair_dj[i], t.pair_di[i], 0, i));
    if (t.pair_di[i] != hr.back().y + hr.back().z) {
      delete c;
      return EVLB_EUNSUPPORTED;
    }
    ++hr.back().z;
    hd.push_back(t.pair_cx[i]);
    hd.push_back(t.pair_cy[i]);
  }
  const int nrow = (int)hr.size();
  hr.resize(L.nrow + ROWPAD, make_int4(0, 0, 0, 0));
  std::vector<int> hi;
  for (size_t i = 0; i < t.avg_w.size(); ++i) hi.push_back(t.avg_dj[i] * PX + t.avg_di[i]);
  double* tabd = (double*)(ws + L.tab_d);
  int4* tabr = (int4*)(ws + L.tab_i);
  int* tabi = (int*)(tabr + L.nrow + ROWPAD);
  // ordered on the caller's stream, which is synchronised before the host
  // vectors go out of scope
  if (nrow > L.nrow ||
      hipMemcpyAsync(tabd, hd.data(), hd.size() * sizeof(double), hipMemcpyHostToDevice, st) != hipSuccess ||
      hipMemcpyAsync(tabr, hr.data(), hr.size() * sizeof(int4), hipMemcpyHostToDevice, st) != hipSuccess ||
      hipMemcpyAsync(tabi, hi.data(), hi.size() * sizeof(int), hipMemcpyHostToDevice, st) != hipSuccess ||
      hipMemsetAsync(ws + L.status, 0, 256, st) != hipSuccess || hipStreamSynchronize(st) != hipSuccess) {
    delete c;
    return EVLB_EHIP;
  }
  c->vel = tabd;
  c->meq = tabd + Q;
  c->dpm = tabd + Q + Q * Q;
  c->avg_w = tabd + Q + 2 * Q * Q;
  c->disc_c = (const dbl2*)(tabd + o_c);
  c->avg_ofs = tabi;
  c->disc_rows = tabr;
  Dev& d = c->dev;
  d.nx = c->nx;
  d.ny = c->ny;
  d.ntot = c->N;
  d.inv_dx = 1.0 / p->dx;
  const double sg = p->sigma;
  d.b = 2.0 * M_PI * sg * sg * sg / 3.0;
  d.eta_c = M_PI * sg * sg * sg / 6.0;
  d.mu0c = 5.0 / (16.0 * sg * sg * std::sqrt(M_PI));
  d.weno_eps = p->weno_eps;
  d.g_ext = p->g_ext;
  d.force_model = p->force_model;
  d.term_mask = p->term_mask;
  d.T_iso = p->T_iso;
  d.navg = L.navg;
  d.npair = p->force_model == EVLB_FORCE_EV1 ? L.npair : 0;
  d.nrow = d.npair > 0 ? nrow : 0;
  d.halo = L.halo;
  d.status = (int*)(ws + L.status);
  *out = c;
  return EVLB_OK;
}

void destroy(Ctx* c) { delete c; }
long long node_count(const Ctx* c) { return c->N; }
const std::vector<double>& velocities(const Ctx* c) { return c->hvel; }
int* status_word(const Ctx* c) { return c->dev.status; }

namespace {

int launched() { return hipGetLastError() == hipSuccess ? EVLB_OK : EVLB_EHIP; }

int launch_raw(Ctx* c, const double* f, hipStream_t st) {
  const unsigned nb = (unsigned)((c->N + MNODES - 1) / MNODES);
  hipLaunchKernelGGL(raw_sums_kernel, dim3(nb), dim3(256), 0, st, c->dev, f, (double*)(c->ws + c->L.raw), c->vel);
  return launched();
}

template <class SH>
int launch_fields_shape(Ctx* c, hipStream_t st) {
  static_assert(SH::FG <= ROWPAD, "the next row of every group exists");
  const dim3 grid((c->nx + SH::TX - 1) / SH::TX, (c->ny + SH::TY - 1) / SH::TY);
  hipLaunchKernelGGL((fields_kernel<SH>), grid, dim3(SH::NT),
                     fields_lds_bytes<SH>(c->L.halo, c->dev.npair, c->L.navg), st, c->dev,
                     (const double*)(c->ws + c->L.raw), (double*)(c->ws + c->L.fld), c->avg_ofs, c->avg_w,
                     c->disc_rows, c->disc_c);
  return launched();
}

int launch_fields(Ctx* c, hipStream_t st) {
  return c->small ? launch_fields_shape<FieldsSmall>(c, st) : launch_fields_shape<FieldsWide>(c, st);
}

template <bool ADV, bool FRC>
void launch_fused(Ctx* c, const FusedArgs& A, dim3 grid, int first, hipStream_t st) {
  if (first)
    hipLaunchKernelGGL((fused_kernel<ADV, FRC, true>), grid, dim3(SNT), 0, st, c->dev, A, c->vel, c->meq, c->dpm);
  else
    hipLaunchKernelGGL((fused_kernel<ADV, FRC, false>), grid, dim3(SNT), 0, st, c->dev, A, c->vel, c->meq, c->dpm);
}

// one evaluation: the fields of the raw sums in the workspace, then
// out = a f0 + b fs + c L(fs) and (want_mom) the raw sums of out
int stage(Ctx* c, const double* fs, const double* f0, double* out, double a, double b, double cc, int first,
          int want_mom, hipStream_t st) {
  int rc = launch_fields(c, st);
  if (rc) return rc;
  const double eps = c->dev.weno_eps;
  FusedArgs A{fs, f0, out, (const double*)(c->ws + c->L.fld), (double*)(c->ws + c->L.raw), a, b, cc, 0.3 * eps,
              0.75 * eps, first, want_mom, c->nstrip, c->seglen};
  const dim3 grid((unsigned)(2 * c->nstrip * c->nseg));
  const bool adv = (c->dev.term_mask & EVLB_TERM_ADV) != 0, frc = (c->dev.term_mask & EVLB_TERM_FORCE) != 0;
  if (adv && frc)
    launch_fused<true, true>(c, A, grid, first, st);
  else if (adv)
    launch_fused<true, false>(c, A, grid, first, st);
  else if (frc)
    launch_fused<false, true>(c, A, grid, first, st);
  else
    launch_fused<false, false>(c, A, grid, first, st);
  return launched();
}

}  // namespace

int set_equilibrium(Ctx* c, const double* n, const double* u, const double* T, double* f, hipStream_t st) {
  const unsigned nb = (unsigned)((c->N + ENODES - 1) / ENODES);
  hipLaunchKernelGGL(equilibrium_kernel, dim3(nb), dim3(256), 0, st, c->dev, n, u, T, f, c->meq);
  return launched();
}

int step(Ctx* c, double* f, int nsteps, hipStream_t st) {
  static const double RKA[3] = {0.0, 0.75, 1.0 / 3.0};
  static const double RKB[3] = {1.0, 0.25, 2.0 / 3.0};
  double* f1 = (double*)(c->ws + c->L.f1);
  double* f2 = (double*)(c->ws + c->L.f2);
  int rc = launch_raw(c, f, st);
  if (rc) return rc;
  const double dt = c->p.dt;
  for (int n = 0; n < nsteps; ++n) {
    for (int s = 0; s < 3; ++s) {
      const double* fs = s == 0 ? f : (s == 1 ? f1 : f2);
      double* W = s == 0 ? f1 : (s == 1 ? f2 : f);  // stage 3 overwrites f^n in place, element by element
      rc = stage(c, fs, f, W, RKA[s], RKB[s], RKB[s] * dt, s == 0, 1, st);
      if (rc) return rc;
    }
  }
  return EVLB_OK;
}

int rhs(Ctx* c, const double* f, double* L, hipStream_t st) {
  int rc = launch_raw(c, f, st);
  if (rc) return rc;
  return stage(c, f, f, L, 0.0, 0.0, 1.0, 1, 0, st);
}

int moments(Ctx* c, const double* f, double* n, double* u, double* T, double* q, hipStream_t st) {
  const unsigned nb = (unsigned)((c->N + MNODES - 1) / MNODES);
  hipLaunchKernelGGL(moments_kernel, dim3(nb), dim3(256), 0, st, c->dev, f, n, u, T, q, c->vel);
  return launched();
}

}  // namespace evlb2d
