// EV-FDLB time step for MI355X (gfx950): fused HIP kernels and the C ABI
// declared in include/evlb.h.
//
// One TVD-RK3 stage is ONE kernel.  A workgroup owns a tile of consecutive
// nodes of one periodic system and all q velocities (phases of the wide tile):
//   1. load     F, G rows of the tile plus a 3-node halo (WENO-5) into LDS;
//               the density window (force / averaged density halo) and
//               u, T (gradient halo) from the moments of the previous stage.
//   2. fields   averaged density and contact value (eq:carnstar, Sec. II A)
//               on the tile +-2; WENO-5 face values of every row.
//   3. fields   Vlasov force (eq:F1 / eq:F2), transport (eq:viscosity,
//               eq:tau, eq:prandtl), J1 gradients (eq:J1) per node.
//   4. update   lanes = nodes, wavefront = group of velocities: Hermite
//               equilibrium, momentum derivative, Shakhov term, J1, advection,
//               RK3 combine; partial velocity moments of the new state.
//   5. reduce   moments (n, u, T, q) of the new state -> global, read by the
//               next stage.
// Global state is structure-of-arrays [2][q][n_tot] (node fastest), so every
// row load and store of a wavefront is one contiguous 512-byte segment.
//
// Tile shapes: wide tiles (64 nodes, groups of velocities per wavefront,
// tables through the scalar cache), narrow and broad tiles (16 and 32 nodes, a
// mirror pair of velocities per lane, the velocity-space contractions on the
// f64 MFMA) for grids too small to fill the chip, and column tiles (one
// wavefront of 63 nodes, a node's whole velocity column in registers) for
// large grids.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "../../include/evlb.h"
#include "evlb2d.h"
#include "resident.h"
#include "tables.h"

namespace {

constexpr int W = 64;          // nodes per tile == lanes of a wavefront
constexpr int HF = 3;          // distribution halo of the WENO-5 faces
constexpr int MS_MAX = 16;     // max sigma/dx
constexpr int MF_MAX = 64;     // max r_cut/dx
constexpr int HN_MAX = MF_MAX; // density window half width
constexpr int NFIELD = 10;

enum { NF_N, NF_U, NF_T, NF_NU, NF_S, NF_PRE, NF_A, NF_B, NF_U1, NF_FX };

// Averaging weights at 0, force taps at TAB_CF, zeros elsewhere.
constexpr int TAB_CF = 2 * MS_MAX + 1, NTAB = TAB_CF + MF_MAX;

struct DevParams {
  const double* vel;   // [q]
  const double* meq;   // [q][q]
  const double* ntab;  // [NTAB] averaging weights and force taps
  const double* pairs; // [q/2][2q] coefficients of a mirror pair (pair_table)
  const double* mx;    // [operands][64] MFMA operands of the mirror shape
  const double* dpm;   // [q][q]
  const double* savg;  // [2 ms + 1]
  const double* cfor;  // [mf]
  const double* cphi;  // [mf] d cfor / d phi_sigma
  const double* csig;  // [mf] d cfor / d sigma
  const double* ssig;  // [2 ms + 1] d savg / d sigma
  const int4* tiles;   // {system offset, system nodes, tile start, 0}
  int ntiles;
  int single;          // one system: tile t starts at node t * width
  int onex;            // small grid: all workgroups on one XCD (grid_index)
  int ms, mf, hn;
  long long ntot;
  double dx, inv_dx, dt;
  double b;        // 2 pi sigma^3 / 3
  double eta_c;    // pi sigma^3 / 6
  double mu0c;     // 5 / (16 sigma^2 sqrt(pi)):  mu0 = mu0c sqrt(T)
  double sigma;
  double weno_eps, weno_e3, weno_e75, g_ext, two_a, kappa;
  double T_iso;    // > 0: isothermal, the temperature the next stage sees
  const double* tiso;  // per node: the isothermal temperature of its system (0 = thermal), or null
  int force_model, term_mask;
  int* status;     // [0] non-finite latch, [1] barrier abort latch
  unsigned* bar;   // [0] arrival count, [1] generation
};

struct StageArgs {
  const double* f_prev;  // f^(s-1)
  const double* f_n;     // f^n (RK3 base)
  double* f_out;         // f^(s), or L(f) in rhs mode
  const double* mom_in;  // [4][ntot] n, u, T, q of f_prev
  double* mom_out;       // [4][ntot] of f_out
  double alpha, beta;    // f_out = alpha f_n + beta (f_prev + dt L)
  int first;             // f_n == f_prev
  int rhs_mode;          // write L(f_prev) instead of a stage
};

// The right-hand-side terms that a kernel is compiled for: all of them, or
// advection and force as in TERMS (0 .. 3) and the collision terms by the
// call's mask, or (ANY_TERMS) every one by the mask.  A term that is off adds
// zeros, not zero times what a node without a density or a temperature gives
// it.
constexpr int ANY_TERMS = -1;
template <int TERMS>
__device__ __forceinline__ bool term_on(const DevParams& P, int bit) {
  if (TERMS == EVLB_TERM_ALL) return true;
  if (TERMS != ANY_TERMS && (bit == EVLB_TERM_ADV || bit == EVLB_TERM_FORCE)) return TERMS & bit;
  return P.term_mask & bit;
}

// 1/x from the hardware reciprocal (within 2^-24.4) and one third-order step r
// <- r (1 + d + d^2), d = 1 - x r: within an ulp or two of the quotient, with
// a shorter dependency chain than the correctly rounded division
__device__ __forceinline__ double rcpn(double x) {
  const double r = __builtin_amdgcn_rcp(x), d = fma(-x, r, 1.0);
  return fma(r, fma(d, d, d), r);
}

// Lane i takes lane i + 1's value across the whole wavefront (DPP wave_shl:1;
// lane 63 gets 0).  Two VALU moves, where a shuffle is an LDS-crossbar round
// trip.
__device__ __forceinline__ double wave_next(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x130, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x130, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (unsigned long long)(unsigned)lo | ((unsigned long long)(unsigned)hi << 32));
}

// Constants of the faces; the plain numbers in scalar registers, for as
// literals the compiler puts them into two-operand fused multiply-adds, each
// behind a register copy.  (Not volatile: behind a volatile statement the
// compiler no longer reads uniform tables through the scalar cache, which
// doubled the wide kernel's registers and time.)
struct WenoK {
  double e3, e75, m275, m125, p25;
};
__device__ __forceinline__ WenoK weno_k(const DevParams& P) {
  WenoK K{P.weno_e3, P.weno_e75, -2.75, -1.25, 2.5};
  asm("" : "+s"(K.m275), "+s"(K.m125), "+s"(K.p25));
  return K;
}

// Classical WENO-5 (Jiang & Shu) face value from the five upwind-ordered
// values v0..v4 = f_{i-2}..f_{i+2}; alpha_r = d_r/(eps+beta_r)^2 combined
// over a common denominator (one reciprocal), in the first differences
// e_m = v_(m+1) - v_m: the candidates less v2 are g0 = (5 e1 -
// 2 e0) / 6, 6 g1 = e1 + 2 e2, 3 g2 = 2 e2 - e3 / 2; three quarters of the
// smoothness indicators are the quadratic forms e0 (e0 - 11/4 e1) + 5/2 e1^2,
// e1 (e1 - 5/4 e2) + e2^2 and e3 (e3 - 11/4 e2) + 5/2 e2^2 (eps enters them
// with 3/4, under the factor 5/2 with 3/10); with the linear weights as 10 d_r
// = (1, 6, 3) the value is v2 plus the normalised weighted corrections.  The
// reciprocal is the hardware's, within 2^-24.4 on this part, and one
// third-order step.  36 instructions.
__device__ __forceinline__ double weno5(double v0, double v1, double v2, double v3, double v4,
                                        const WenoK& K) {
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

// Launch shape of the wide stage kernel: tiles of W = 64 nodes, NG groups of
// velocities (thread = node j x group g, NT = W * NG threads).  A velocity
// group is uniform over a wavefront, so the constant tables are read through
// the scalar cache.  (The mirror shapes of 16 and 32 nodes have their
// own tile function.)
template <int Q, int W, int NG>
struct Shape {
  static constexpr int NT = W * NG;
  static constexpr int VPT = Q / NG;
  static_assert(W % 64 == 0, "a velocity group spans whole wavefronts");
  static_assert(Q % NG == 0, "velocity groups must divide q");
  static_assert(NG >= 2, "two node groups are needed for the field phase");
  static_assert(NT <= 1024, "workgroup too large");
};

template <int Q, int W, int NG>
struct Smem {
  double f[2 * Q][W + 2 * HF];     // F rows then G rows, tile + WENO halo
  union {
    double flux[2 * Q][W + 1];     // WENO-5 face values
    double red[NG][6][W];          // partial velocity moments
  };
  double n[W + 2 * HN_MAX];        // density window
  double u[W + 4], T[W + 4], X[W + 4], chi[W + 4];
  double a[Q][W];                  // Hermite moments of the local Maxwellian
  union {
    double fpart[NG][W];           // partial force sums
    double msum[6][W];             // velocity moments of the new state
  };
  double nf[NFIELD][W];
  double sav[2 * MS_MAX + 1];      // averaging weights
  double cf[MF_MAX];               // EV1 force taps
};

// i mod n for indices at most 128 beyond either end; the loops only for the
// systems smaller than that (n is uniform: a scalar branch), whose windows
// wrap more than once.  The loops alone, two branches on the execution mask
// each, cost 3% of a small stage (4.06 -> 3.92 us) and 2% of a middling one.
__device__ __forceinline__ int wrapi(int i, int n) {
  i += i < 0 ? n : 0;
  i -= i >= n ? n : 0;
  if (n < 128) {
    while (i < 0) i += n;
    while (i >= n) i -= n;
  }
  return i;
}

// The averaging weights and force taps into LDS.  All loads are issued
// before the first LDS write, so the copy costs one memory round trip.
template <int Q, int W, int NG>
__device__ __forceinline__ void load_tables(const DevParams& P, Smem<Q, W, NG>& S) {
  constexpr int NT = Shape<Q, W, NG>::NT;
  constexpr int NSAV = 2 * MS_MAX + 1;
  constexpr int NALL = NSAV + MF_MAX;
  constexpr int L = (NALL + NT - 1) / NT;
  const int tid = threadIdx.x;
  double v[L];
#pragma unroll
  for (int i = 0; i < L; ++i) {
    const int e = tid + i * NT;
    // one load per entry through a selected pointer (separate loads in the
    // branches would be serialised by the register they share)
    const double* src = nullptr;
    int si = 0;
    if (e < 2 * P.ms + 1) { src = P.savg; si = e; }
    else if (e >= NSAV && e < NSAV + P.mf) { src = P.cfor; si = e - NSAV; }
    v[i] = src ? src[si] : 0.0;
  }
#pragma unroll
  for (int i = 0; i < L; ++i) {
    const int e = tid + i * NT;
    if (e < NSAV) S.sav[e] = v[i];
    else if (e < NALL) S.cf[e - NSAV] = v[i];
  }
  __syncthreads();
}

// One stage over one tile (see file header).
template <int Q, int W, int NG>
__device__ void stage_tile(const DevParams& P, const StageArgs& A, int tile, Smem<Q, W, NG>& S) {
  using SH = Shape<Q, W, NG>;
  constexpr int NT = SH::NT;
  constexpr int VPT = SH::VPT;
  const int tid = threadIdx.x;
  const int4 td = P.tiles[tile];
  const int off = td.x, nsys = td.y, i0 = td.z;
  const long long ntot = P.ntot;
  const int hn = P.hn;
  const int j = tid % W;
  const int g = __builtin_amdgcn_readfirstlane(tid / W);
  const int kbase = g * VPT;
  const bool valid = (i0 + j) < nsys;
  const long long gnode = off + i0 + j;

  // ---- 1. load ----------------------------------------------------------
  // RK3 base values of this thread's velocities, fetched first so that their
  // latency overlaps the tile staging
  double Fn[VPT], Gn[VPT];
  const bool need_base = !A.first && !A.rhs_mode && valid;
#pragma unroll
  for (int v = 0; v < VPT; ++v) {
    Fn[v] = 0.0;
    Gn[v] = 0.0;
    if (need_base) {
      Fn[v] = A.f_n[(long long)(kbase + v) * ntot + gnode];
      Gn[v] = A.f_n[(long long)(Q + kbase + v) * ntot + gnode];
    }
  }
  // tile + WENO halo of F and G, the density window, u and T on the tile +-2:
  // every load is issued before the first LDS write (one round trip)
  constexpr int FW = W + 2 * HF;
  constexpr int NFV = 2 * Q * FW;
  constexpr int LF = (NFV + NT - 1) / NT;
  double fv[LF];
#pragma unroll
  for (int i = 0; i < LF; ++i) {
    const int idx = tid + i * NT;
    fv[i] = 0.0;
    if (idx < NFV) {
      const int r = idx / FW;
      const int c = idx - r * FW;
      fv[i] = A.f_prev[(long long)r * ntot + off + wrapi(i0 - HF + c, nsys)];
    }
  }
  const double* mn = A.mom_in;
  constexpr int LN = (W + 2 * HN_MAX + NT - 1) / NT;
  const int nwin = W + 2 * hn;
  double nv[LN];
#pragma unroll
  for (int i = 0; i < LN; ++i) {
    const int c = tid + i * NT;
    nv[i] = 0.0;
    if (c < nwin) nv[i] = mn[off + wrapi(i0 - hn + c, nsys)];
  }
  static_assert(NT >= W + 4, "one thread per node of the tile +-2");
  double uv = 0.0, Tv = 0.0;
  if (tid < W + 4) {
    const int node = off + wrapi(i0 - 2 + tid, nsys);
    uv = mn[ntot + node];
    Tv = mn[2 * ntot + node];
  }
  double qj = 0.0;
  if (tid >= W && tid < 2 * W) qj = mn[3 * ntot + off + wrapi(i0 + j, nsys)];
  // isothermal temperature of the own node's system, read with the tile
  double tiso = P.T_iso;
  if (P.tiso && tid < W && valid) tiso = P.tiso[gnode];
#pragma unroll
  for (int i = 0; i < LF; ++i) {
    const int idx = tid + i * NT;
    if (idx < NFV) {
      const int r = idx / FW;
      S.f[r][idx - r * FW] = fv[i];
    }
  }
#pragma unroll
  for (int i = 0; i < LN; ++i) {
    const int c = tid + i * NT;
    if (c < nwin) S.n[c] = nv[i];
  }
  if (tid < W + 4) {
    S.u[tid] = uv;
    S.T[tid] = Tv;
  }
  __syncthreads();

  // ---- 2. contact value, Hermite moments, force partial sums, WENO faces ---
  {
    // contact value chi(nbar) and X = n^2 chi T on the tile +-2
    for (int c = tid; c < W + 4; c += NT) {
      const int cn = c + hn - 2;
      double s0 = 0.0, s1 = 0.0;
      int jj = -P.ms;
      for (; jj + 1 <= P.ms; jj += 2) {
        s0 += S.sav[jj + P.ms] * S.n[cn + jj];
        s1 += S.sav[jj + 1 + P.ms] * S.n[cn + jj + 1];
      }
      if (jj <= P.ms) s0 += S.sav[jj + P.ms] * S.n[cn + jj];
      const double eta = P.eta_c * (s0 + s1);
      const double om = 1.0 - eta;
      const double chi = (2.0 - eta) / (2.0 * om * om * om);
      const double nn = S.n[cn];
      S.chi[c] = chi;
      S.X[c] = nn * nn * chi * S.T[c];
    }
    // Hermite moments a_0 = n, a_1 = n u, a_{l+1} = u a_l + l (T - 1) a_{l-1}
    if (tid >= NT - W) {
      const int jn = tid - (NT - W);
      const double n = S.n[jn + hn], u = S.u[jn + 2], tm1 = S.T[jn + 2] - 1.0;
      double am = n, a = n * u;
      S.a[0][jn] = am;
      S.a[1][jn] = a;
#pragma unroll
      for (int l = 1; l < Q - 1; ++l) {
        const double an = u * a + (double)l * tm1 * am;
        am = a;
        a = an;
        S.a[l + 1][jn] = a;
      }
    }
    // EV1 force: node j, chunk g of the paired taps
    if (P.force_model == EVLB_FORCE_EV1) {
      const int ch = (P.mf + NG - 1) / NG;
      const int m0 = 1 + g * ch;
      const int m1 = min(P.mf, m0 + ch - 1);
      const int cn = j + hn;
      double s0 = 0.0, s1 = 0.0;
      int m = m0;
      for (; m + 1 <= m1; m += 2) {
        s0 += S.cf[m - 1] * (S.n[cn + m] - S.n[cn - m]);
        s1 += S.cf[m] * (S.n[cn + m + 1] - S.n[cn - m - 1]);
      }
      if (m <= m1) s0 += S.cf[m - 1] * (S.n[cn + m] - S.n[cn - m]);
      S.fpart[g][j] = s0 + s1;
    }
    if (P.term_mask & EVLB_TERM_ADV) {
      const WenoK K = weno_k(P);
      for (int idx = tid; idx < 2 * Q * (W + 1); idx += NT) {
        const int r = idx / (W + 1);
        const int jf = idx - r * (W + 1);      // face i0 + jf - 1/2
        const int k = r < Q ? r : r - Q;
        const bool pos = k >= Q / 2;             // p_k > 0: upwind from the left
        const double* fr = &S.f[r][0];
        const int b0 = pos ? jf : jf + 5;
        const int st = pos ? 1 : -1;
        S.flux[r][jf] = weno5(fr[b0], fr[b0 + st], fr[b0 + 2 * st], fr[b0 + 3 * st], fr[b0 + 4 * st], K);
      }
    }
  }
  __syncthreads();

  // ---- 3. node fields: force and gradients (group 0), transport (group 1) --
  if (tid < W) {
    const int c = j + 2;
    const int cn = j + hn;
    const double idx12 = P.inv_dx * (1.0 / 12.0);
    double Fx = P.g_ext;
    if (P.force_model == EVLB_FORCE_EV1) {
      double s = 0.0;
#pragma unroll
      for (int gg = 0; gg < NG; ++gg) s += S.fpart[gg][j];
      Fx += s;
    } else if (P.force_model == EVLB_FORCE_EV2) {
      const double d1 = (S.n[cn - 2] - 8.0 * S.n[cn - 1] + 8.0 * S.n[cn + 1] - S.n[cn + 2]) * idx12;
      const double d3 = (-S.n[cn - 2] + 2.0 * S.n[cn - 1] - 2.0 * S.n[cn + 1] + S.n[cn + 2]) *
                        (0.5 * P.inv_dx * P.inv_dx * P.inv_dx);
      Fx += P.two_a * d1 + P.kappa * d3;
    }
    const double T = S.T[c];
    S.nf[NF_A][j] = (S.X[c - 2] - 8.0 * S.X[c - 1] + 8.0 * S.X[c + 1] - S.X[c + 2]) * idx12 / S.X[c];
    S.nf[NF_B][j] = (S.T[c - 2] - 8.0 * S.T[c - 1] + 8.0 * S.T[c + 1] - S.T[c + 2]) * idx12 / T;
    S.nf[NF_U1][j] = (S.u[c - 2] - 8.0 * S.u[c - 1] + 8.0 * S.u[c + 1] - S.u[c + 2]) * idx12;
    S.nf[NF_FX][j] = Fx;
    S.nf[NF_N][j] = S.n[cn];
    S.nf[NF_U][j] = S.u[c];
    S.nf[NF_T][j] = T;
  } else if (tid < 2 * W) {
    // transport: mu (eq:viscosity), tau (eq:tau), Pr (eq:prandtl); rate chi/tau
    const int c = j + 2;
    const double n = S.n[j + hn];
    const double T = S.T[c];
    const double chi = S.chi[c];
    const double bn = P.b * n;
    const double y = bn * chi;
    const double mu0 = P.mu0c * sqrt(T);
    const double c12 = 0.16 * (1.0 + 12.0 / M_PI);
    const double c32 = 0.36 * (1.0 + 32.0 / (9.0 * M_PI));
    const double mu = mu0 * (1.0 / chi + 0.8 * bn + c12 * bn * bn * chi);
    S.nf[NF_NU][j] = chi * n * T * (1.0 + 0.4 * y) / mu;
    const double Pr = (2.0 / 3.0) * (1.0 + 0.6 * y) * (1.0 + 0.8 * y + c12 * y * y) /
                      ((1.0 + 0.4 * y) * (1.0 + 1.2 * y + c32 * y * y));
    S.nf[NF_S][j] = (1.0 - Pr) * qj / (5.0 * n * T * T);
    S.nf[NF_PRE][j] = -bn * chi;
  }
  __syncthreads();

  // ---- 4. update -----------------------------------------------------------
  const double* meq = P.meq;
  const double* dpm = P.dpm;
  const double* vel = P.vel;
  double pm[6] = {0, 0, 0, 0, 0, 0};
  {
    const double u = S.nf[NF_U][j], T = S.nf[NF_T][j];
    const double nu = S.nf[NF_NU][j], sS = S.nf[NF_S][j], pre = S.nf[NF_PRE][j];
    const double Ag = S.nf[NF_A][j], Bg = S.nf[NF_B][j], Ug = S.nf[NF_U1][j];
    const double Fx = S.nf[NF_FX][j];
    const double invT = 1.0 / T;
    // Hermite equilibrium E_k = sum_l meq[k][l] a_l
    double E[VPT];
#pragma unroll
    for (int v = 0; v < VPT; ++v) E[v] = 0.0;
#pragma unroll
    for (int l = 0; l < Q; ++l) {
      const double al = S.a[l][j];
#pragma unroll
      for (int v = 0; v < VPT; ++v) E[v] += meq[(kbase + v) * Q + l] * al;
    }
    // momentum derivative (Dp F)_k, (Dp G)_k
    double dF[VPT], dG[VPT];
#pragma unroll
    for (int v = 0; v < VPT; ++v) { dF[v] = 0.0; dG[v] = 0.0; }
    if (P.term_mask & EVLB_TERM_FORCE) {
#pragma unroll
      for (int kp = 0; kp < Q; ++kp) {
        const double fk = S.f[kp][j + HF];
        const double gk = S.f[Q + kp][j + HF];
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
          const double d = dpm[(kbase + v) * Q + kp];
          dF[v] += d * fk;
          dG[v] += d * gk;
        }
      }
    }
#pragma unroll
    for (int v = 0; v < VPT; ++v) {
      const int k = kbase + v;
      const double pk = vel[k];
      const double F = S.f[k][j + HF];
      const double G = S.f[Q + k][j + HF];
      const double xi = pk - u;
      const double th = xi * xi * invT;
      double LF = 0.0, LG = 0.0;
      if (P.term_mask & EVLB_TERM_ADV) {
        LF = -pk * (S.flux[k][j + 1] - S.flux[k][j]) * P.inv_dx;
        LG = -pk * (S.flux[Q + k][j + 1] - S.flux[Q + k][j]) * P.inv_dx;
      }
      if (P.term_mask & EVLB_TERM_FORCE) {
        LF -= Fx * dF[v];
        LG -= Fx * dG[v];
      }
      if (P.term_mask & EVLB_TERM_J0) {
        const double FS = E[v] * (1.0 + sS * xi * (th - 3.0));
        const double GS = T * E[v] * (1.0 + sS * xi * (th - 1.0));
        LF -= nu * (F - FS);
        LG -= nu * (G - GS);
      }
      if (P.term_mask & EVLB_TERM_J1) {
        LF += pre * E[v] * (xi * (Ag + 0.3 * (th - 3.0) * Bg) + 0.6 * (th - 1.0) * Ug);
        LG += pre * T * E[v] * (xi * (Ag + 0.3 * (th - 1.0) * Bg) + 0.2 * (3.0 * th - 1.0) * Ug);
      }
      double Fo, Go;
      if (A.rhs_mode) {
        Fo = LF;
        Go = LG;
      } else {
        const double Fb = A.first ? F : Fn[v];
        const double Gb = A.first ? G : Gn[v];
        Fo = A.alpha * Fb + A.beta * (F + P.dt * LF);
        Go = A.alpha * Gb + A.beta * (G + P.dt * LG);
      }
      if (valid) {
        A.f_out[(long long)k * ntot + gnode] = Fo;
        A.f_out[(long long)(Q + k) * ntot + gnode] = Go;
      }
      const double p2 = pk * pk;
      pm[0] += Fo;
      pm[1] += pk * Fo;
      pm[2] += p2 * Fo;
      pm[3] += p2 * pk * Fo;
      pm[4] += Go;
      pm[5] += pk * Go;
    }
  }
  __syncthreads();  // faces (aliased by red) fully consumed
  if (A.rhs_mode) return;
#pragma unroll
  for (int m = 0; m < 6; ++m) S.red[g][m][j] = pm[m];
  __syncthreads();

  // ---- 5. moments of the new state --------------------------------------
  for (int t = tid; t < 6 * W; t += NT) {
    const int m = t / W, jj = t - m * W;
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int gg = 0; gg + 1 < NG; gg += 2) {
      s0 += S.red[gg][m][jj];
      s1 += S.red[gg + 1][m][jj];
    }
    if (NG & 1) s0 += S.red[NG - 1][m][jj];
    S.msum[m][jj] = s0 + s1;
  }
  __syncthreads();
  if (tid < W && valid) {
    const double n = S.msum[0][tid];
    const double u = S.msum[1][tid] / n;
    const double T = (2.0 / 3.0) * (0.5 * S.msum[2][tid] + S.msum[4][tid] - 0.5 * n * u * u) / n;
    const double x3 = S.msum[3][tid] - 3.0 * u * S.msum[2][tid] + 3.0 * u * u * S.msum[1][tid] - u * u * u * n;
    const double q = 0.5 * x3 + S.msum[5][tid] - u * S.msum[4][tid];
    A.mom_out[gnode] = n;
    A.mom_out[ntot + gnode] = u;
    A.mom_out[2 * ntot + gnode] = tiso > 0.0 ? tiso : T;
    A.mom_out[3 * ntot + gnode] = q;
    if (!(n > 0.0) || !(T > 0.0) || !isfinite(n) || !isfinite(T) || !isfinite(q) || !isfinite(u))
      P.status[0] = 1;
  }
  __syncthreads();
}

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int WN = 16;  // nodes per narrow tile

// ---------------------------------------------------------------------------
// Mirror shape: a tile of W nodes, wavefronts of column groups and four node
// wavefronts.  A column wavefront takes NC = 128 / Q neighbouring nodes (Q = 24:
// 4) of one distribution; its lane holds a mirror pair of velocities (r, Q - 1 -
// r) of one node, p_(Q-1-r) = -p_r, in the layout of v_mfma_f64_4x4x4 (four
// blocks b = L >> 2 & 3 of four columns L & 3 by four contraction indices or
// rows k = L >> 4; an A operand has its row in L & 3): r = KT k + kt with KT = Q /
// 8 and kt the block's part of r (Q = 8: the blocks are four column groups; Q =
// 16: two column groups by kt; Q = 24: kt = b, the fourth block idle).  Both
// contractions split into even and odd halves over mirror pairs, (Q / 2) x (Q /
// 2) each, straight from the registers:
//   (Dp f)_r, (Dp f)_(Q-1-r) = o +- e,  e = S (f_j + f_(Q-1-j)), o = A (f_j - f_(Q-1-j)),
//   E_r, E_(Q-1-r) = e +- o,            e, o = sums over the even and odd Hermite moments,
// and the velocity sums of the new state are the moments sum p^i f, i < 4, of
// each distribution, a 4 x Q product.  Four node wavefronts work beside the
// columns.  Phases (a barrier between):
//   load      f with a 3-node halo, density window, u, T, tables to LDS
//   faces     columns: the upwind face of each value, Dp f; nodes: 0 contact
//             value, 1 Hermite moments, 2 force, 3 the tile's edge faces
//   node      columns: equilibrium, the other face from LDS; nodes: 0 gradients
//             and J1, 1 force, 2 transport and J0
//   update    new values, their store, their moments
//   moments   n, u, T, q of the new state
// A stage is a chain of latencies at small grids and bound by vector
// instructions and occupancy at large ones.  The node wavefronts' chains are
// the longest of the two middle phases, so they issue first (s_setprio: 1 to
// 4%).  A stage of 16-node tiles in a captured graph, where an empty launch is
// 1.6 us, against one value per thread, full 16x16x4 products and the partial
// velocity moments through LDS:
//   256 nodes   q 8 5.93 -> 3.40   q 16 5.85 -> 3.44   q 24 6.24 -> 4.07 us
// (with the loads' side of it on one XCD, see grid_index, and the leading
// arguments preloaded, see stage_kernel_mirror; 3.68, 3.92 and 4.54 without; the
// terms known at compile time, see launch_stage_mirror).
// ---------------------------------------------------------------------------
template <int Q, int W>
struct Mirror {
  static constexpr int KT = Q / 8;                         // parts of r
  static constexpr int NC = Q == 24 ? 4 : 128 / Q;         // nodes per column wavefront
  static constexpr int NR = Q == 8 ? 1 : (Q == 16 ? 2 : 4);  // blocks that hold parts of r
  static constexpr int NCW = 2 * (W / NC);                 // column wavefronts
  static constexpr int NT = 64 * (NCW + 4);
  static constexpr int NOP = 4 * NR + 2;                   // MFMA operands per lane
  // row stride in LDS: the lanes of a half wavefront, NC columns of 32 / NC
  // consecutive r, on distinct banks: NC (mod 2 NC) or its negative, at least W + 7
  static constexpr int stride() {
    int s = W + 2 * HF + 1;
    while (s % (Q == 24 ? 8 : 32) != (Q == 24 ? 4 : (Q == 8 ? 16 : 8)) && (Q != 16 || s % 32 != 24)) ++s;
    return s;
  }
  static constexpr int FS = stride();
  static_assert(W % NC == 0 && 64 % W == 0 && W + 4 <= 64 && NT <= 1024, "tile shape");
};

// Per-node quantities of the update, scaled by the stage's factor of L: u, the
// factor of f, force, then per distribution the J1 part of the cubic (4) and
// the J0 part of its coefficients 0, 1 and 3.
enum { MC_U, MC_NUB, MC_FX, MC_F, MC_G = MC_F + 7, NMC = MC_G + 7 };

template <int Q, int W>
struct SmemM {
  double f[2 * Q][Mirror<Q, W>::FS];     // F rows then G rows: node i at i + 3
  double flux[2 * Q][Mirror<Q, W>::FS];  // faces: left of node i at i
  double n[W + 2 * HN_MAX];              // density window
  double u[W + 4], T[W + 4], X[W + 4], chi[W + 4];
  double a[Q][W];                        // Hermite moments of the local Maxwellian
  double fp[64 / W][W];                 // parts of the force
  double co[NMC][W];                     // node coefficients of the update
  double mom[2][4][W];                   // moments of the new F and G
  double tab[NTAB];                      // averaging weights and force taps
  double op[Mirror<Q, W>::NOP][64];      // MFMA operands
};

// lane i takes the value of lane i - 4 S of its 16-lane row (cyclic)
template <int S>
__device__ __forceinline__ double row_rot(double v) {
  if constexpr (S == 0) {
    return v;
  } else {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x120 + 4 * S, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x120 + 4 * S, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (unsigned long long)(unsigned)lo | ((unsigned long long)(unsigned)hi << 32));
  }
}

__device__ __forceinline__ double mfma4(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// sum over the blocks that hold parts of r of (operand s) x (value of the
// block s away)
template <int Q>
__device__ __forceinline__ double mirror_dot(const double* op, double v) {  // op: 64 apart
  double x = mfma4(op[0], v, 0.0);
  if constexpr (Q == 16) {
    x = mfma4(op[64], row_rot<2>(v), x);
  } else if constexpr (Q == 24) {
    x = mfma4(op[64], row_rot<1>(v), x);
    x = mfma4(op[128], row_rot<2>(v), x);
    x = mfma4(op[192], row_rot<3>(v), x);
  }
  return x;
}

template <int Q>
__device__ __forceinline__ double mirror_blocks(double v) {  // sum over the blocks' parts
  if constexpr (Q == 8) return v;
  v += row_rot<2>(v);
  if constexpr (Q == 24) v += row_rot<1>(v);
  return v;
}

template <int Q, int W, int TERMS>
__device__ void stage_tile_mirror(const DevParams& P, const StageArgs& A, int tile, SmemM<Q, W>& S) {
  using M = Mirror<Q, W>;
  constexpr int NT = M::NT, KT = M::KT, NC = M::NC, NR = M::NR, NCW = M::NCW, FS = M::FS;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int off, nsys, i0;
  if (P.single) {
    off = 0;
    nsys = (int)P.ntot;
    i0 = tile * W;
  } else {
    const int4 td = P.tiles[tile];
    off = td.x;
    nsys = td.y;
    i0 = td.z;
  }
  const long long ntot = P.ntot;
  const int hn = P.hn;
  const bool adv = term_on<TERMS>(P, EVLB_TERM_ADV), frc = term_on<TERMS>(P, EVLB_TERM_FORCE);
  const bool j0 = term_on<TERMS>(P, EVLB_TERM_J0), j1 = term_on<TERMS>(P, EVLB_TERM_J1);
  // ---- load: one batch of global loads, then the LDS writes ----------------
  // rows of f: LPR lanes a row, NT / LPR rows at a time
  constexpr int FW = W + 2 * HF, LPR = FW <= 32 ? 32 : 64, RPB = NT / LPR, LF = (2 * Q + RPB - 1) / RPB;
  static_assert(FW <= LPR && NT % LPR == 0, "a row's columns fit its lanes");
  const int fcol = tid % LPR, frow = tid / LPR;
  const double* fsrc = A.f_prev + (long long)frow * ntot + off + wrapi(i0 - HF + fcol, nsys);
  double fv[LF];
#pragma unroll
  for (int i = 0; i < LF; ++i) {
    fv[i] = 0.0;
    if (fcol < FW && frow + i * RPB < 2 * Q) fv[i] = fsrc[(long long)(i * RPB) * ntot];
  }
  const double* mn = A.mom_in;
  constexpr int LN = (W + 2 * HN_MAX + NT - 1) / NT;
  const int nwin = W + 2 * hn;
  double nv[LN];
#pragma unroll
  for (int i = 0; i < LN; ++i) {
    const int c = tid + i * NT;
    nv[i] = 0.0;
    if (c < nwin) nv[i] = mn[off + wrapi(i0 - hn + c, nsys)];
  }
  constexpr int LO = (64 * M::NOP + NT - 1) / NT;
  double ov[LO];
#pragma unroll
  for (int i = 0; i < LO; ++i) {
    ov[i] = 0.0;
    if (tid + i * NT < 64 * M::NOP) ov[i] = P.mx[tid + i * NT];
  }
  // the other arguments into scalar registers before the first branch: one
  // round trip, behind those loads, instead of one at each first use
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::"s"(P.vel), "s"(P.ntab), "s"(P.status), "s"(P.ms), "s"(P.mf), "s"(P.force_model),
               "s"(P.term_mask));
  asm volatile("" ::"s"(P.inv_dx), "s"(P.dt), "s"(P.b), "s"(P.eta_c), "s"(P.mu0c), "s"(P.weno_e3), "s"(P.weno_e75),
               "s"(P.g_ext), "s"(P.two_a), "s"(P.kappa), "s"(P.T_iso), "s"(P.tiso));
  asm volatile("" ::"s"(A.f_n), "s"(A.f_out), "s"(A.mom_out), "s"(A.alpha), "s"(A.beta), "s"(A.first),
               "s"(A.rhs_mode));
  // out = ca f_n + bb f + cc L(f)
  const double cc = A.rhs_mode ? 1.0 : A.beta * P.dt;
  const double ca = A.rhs_mode || A.first ? 0.0 : A.alpha;
  const double bb = A.rhs_mode ? 0.0 : (A.first ? A.alpha + A.beta : A.beta);

  const WenoK K = weno_k(P);
  // node wavefront 0: the tables; 1: u and T of the tile +-2; 2: q of its nodes
  constexpr int LT = (NTAB + 63) / 64;
  double uv, Tv, qv, tv[LT];
  if (wave == NCW) {
#pragma unroll
    for (int i = 0; i < LT; ++i)
      if (lane + 64 * i < NTAB) tv[i] = P.ntab[lane + 64 * i];
  } else if (wave == NCW + 1) {
    if (lane < W + 4) {
      const int node = off + wrapi(i0 - 2 + lane, nsys);
      uv = mn[ntot + node];
      Tv = mn[2 * ntot + node];
    }
  } else if (wave == NCW + 2 && lane < W) {
    qv = mn[3 * ntot + off + wrapi(i0 + lane, nsys)];
  }
  // a column wavefront's f_n
  const int d = wave & 1;
  const int kt = Q == 8 ? 0 : (Q == 16 ? (lane >> 3) & 1 : (lane >> 2) & 3);
  const bool live = kt < KT;  // Q = 24: the fourth block has no velocities
  const int r = KT * (lane >> 4) + (live ? kt : 0);
  const int cw = lane & (NC - 1), c = (wave >> 1) * NC + cw;  // node of a column lane
  const int row0 = d * Q + r, row1 = d * Q + Q - 1 - r;
  const bool valid = live && i0 + c < nsys;
  const long long gnode = off + i0 + c;
  double Fn0, Fn1, pr;
  if (wave < NCW) {
    Fn0 = 0.0;
    Fn1 = 0.0;
    pr = P.vel[r];
    if (!A.first && !A.rhs_mode && valid) {
      Fn0 = A.f_n[(long long)row0 * ntot + gnode];
      Fn1 = A.f_n[(long long)row1 * ntot + gnode];
    }
  }
  // isothermal temperature of the own node's system (moment threads)
  double tiso = P.T_iso;
  if (P.tiso && tid < W && i0 + tid < nsys) tiso = P.tiso[off + i0 + tid];
#pragma unroll
  for (int i = 0; i < LF; ++i)
    if (fcol < FW && frow + i * RPB < 2 * Q) S.f[frow + i * RPB][fcol] = fv[i];
#pragma unroll
  for (int i = 0; i < LN; ++i) {
    const int w = tid + i * NT;
    if (w < nwin) S.n[w] = nv[i];
  }
#pragma unroll
  for (int i = 0; i < LO; ++i)
    if (tid + i * NT < 64 * M::NOP) (&S.op[0][0])[tid + i * NT] = ov[i];
  if (wave == NCW) {
#pragma unroll
    for (int i = 0; i < LT; ++i)
      if (lane + 64 * i < NTAB) S.tab[lane + 64 * i] = tv[i];
  } else if (wave == NCW + 1 && lane < W + 4) {
    S.u[lane] = uv;
    S.T[lane] = Tv;
  }
  __syncthreads();

  // ---- faces, Dp f; contact value and transport; Hermite moments; force ----
  double f0, f1, lf0, lf1, g0, g1;  // column wavefronts
  double nn, chi;                         // node wavefront 0, node lane - 2
  const double* op = &S.op[0][lane];
  // force of node lane % W, share `part` of 64 / W of the paired taps
  auto force_part = [&](int part) {
    constexpr int NP = 64 / W;
    const int j = lane % W;
    const double* nc = &S.n[j + hn];
    double s0 = 0.0, s1 = 0.0;
    if (P.force_model == EVLB_FORCE_EV1) {
      const double* cf = &S.tab[TAB_CF - 1];
      int m = 1 + part;
      for (; m + 4 * NP <= P.mf; m += 5 * NP) {
        s0 += cf[m] * (nc[m] - nc[-m]);
        s1 += cf[m + NP] * (nc[m + NP] - nc[-m - NP]);
        s0 += cf[m + 2 * NP] * (nc[m + 2 * NP] - nc[-m - 2 * NP]);
        s1 += cf[m + 3 * NP] * (nc[m + 3 * NP] - nc[-m - 3 * NP]);
        s0 += cf[m + 4 * NP] * (nc[m + 4 * NP] - nc[-m - 4 * NP]);
      }
      for (; m <= P.mf; m += NP) s0 += cf[m] * (nc[m] - nc[-m]);
    } else if (P.force_model == EVLB_FORCE_EV2 && part == 0) {
      const double idx12 = P.inv_dx * (1.0 / 12.0);
      const double d1 = (nc[-2] - 8.0 * nc[-1] + 8.0 * nc[1] - nc[2]) * idx12;
      const double d3 = (-nc[-2] + 2.0 * nc[-1] - 2.0 * nc[1] + nc[2]) * (0.5 * P.inv_dx * P.inv_dx * P.inv_dx);
      s0 = P.two_a * d1 + P.kappa * d3;
    }
    S.fp[part][j] = s0 + s1;
  };
  if (wave >= NCW) __builtin_amdgcn_s_setprio(2);
  if (wave < NCW) {
    // p_r < 0: the face on the right, upwind from the right; Q - 1 - r: on the left
    const double* x0 = &S.f[row0][c + 2];
    const double* x1 = &S.f[row1][c];
    f0 = x0[1];
    f1 = x1[3];
    g0 = 0.0;
    g1 = 0.0;
    if (adv) {
      lf0 = weno5(x0[4], x0[3], x0[2], x0[1], x0[0], K);
      lf1 = weno5(x1[0], x1[1], x1[2], x1[3], x1[4], K);
      S.flux[row0][c + 1] = lf0;
      S.flux[row1][c] = lf1;
    }
    if (frc) {
      const double e = mirror_dot<Q>(op, f0 + f1), o = mirror_dot<Q>(op + 64 * NR, f0 - f1);
      g0 = o + e;
      g1 = o - e;
    }
  } else if (wave == NCW) {
    if (lane < W + 4) {
      // chi(nbar) and X = n^2 chi T (eq:carnstar); the averaging weights are
      // even: pairs, four in flight
      const double* nc = &S.n[lane + hn - 2];
      const double* sw = &S.tab[P.ms];
      nn = nc[0];
      double s0 = sw[0] * nn, s1 = 0.0;
      int j = 1;
      for (; j + 3 <= P.ms; j += 4) {
        s0 += sw[j] * (nc[j] + nc[-j]);
        s1 += sw[j + 1] * (nc[j + 1] + nc[-j - 1]);
        s0 += sw[j + 2] * (nc[j + 2] + nc[-j - 2]);
        s1 += sw[j + 3] * (nc[j + 3] + nc[-j - 3]);
      }
      for (; j <= P.ms; ++j) s0 += sw[j] * (nc[j] + nc[-j]);
      const double eta = P.eta_c * (s0 + s1);
      const double om = 1.0 - eta;
      chi = (2.0 - eta) * rcpn(2.0 * om * om * om);
      S.chi[lane] = chi;
      S.X[lane] = nn * nn * chi * S.T[lane];
    }
  } else if (wave == NCW + 1) {
    if (lane < W) {
      // Hermite moments a_0 = n, a_1 = n u, a_{l+1} = u a_l + l (T - 1) a_{l-1}
      if (j0 || j1) {
        const double n = S.n[lane + hn], u = S.u[lane + 2], tm1 = S.T[lane + 2] - 1.0;
        double am = n, a = n * u;
        S.a[0][lane] = am;
        S.a[1][lane] = a;
#pragma unroll
        for (int l = 1; l < Q - 1; ++l) {
          const double an = fma(u, a, (double)l * tm1 * am);
          am = a;
          a = an;
          S.a[l + 1][lane] = a;
        }
      } else {
        for (int l = 0; l < Q; ++l) S.a[l][lane] = 0.0;
      }
    }
  } else if (wave == NCW + 2) {
    force_part(lane / W);
  } else if (adv && lane < 2 * Q) {
    // the face of each row that no node's lane forms: right of the last
    // node (p_k > 0) or left of the first
    const bool pos = lane % Q >= Q / 2;
    const double* x = &S.f[lane][pos ? W : 1];
    const double v[5] = {x[0], x[1], x[2], x[3], x[4]};
    S.flux[lane][pos ? W : 0] = weno5(pos ? v[0] : v[4], pos ? v[1] : v[3], v[2], pos ? v[3] : v[1],
                                            pos ? v[4] : v[0], K);
  }
  __syncthreads();

  // ---- equilibrium and the other faces; coefficients per node --------------
  double E0, E1, acc0, acc1;
  if (wave < NCW) {
    acc0 = 0.0;
    acc1 = 0.0;
    const double ev = S.a[2 * r][c], od = S.a[2 * r + 1][c];
    if (adv) {
      const double cpx = cc * P.inv_dx * fabs(pr);
      acc0 = cpx * (lf0 - S.flux[row0][c]);
      acc1 = cpx * (lf1 - S.flux[row1][c + 1]);
    }
    acc0 = fma(ca, Fn0, acc0);
    acc1 = fma(ca, Fn1, acc1);
    const double e = mirror_dot<Q>(op + 128 * NR, ev), o = mirror_dot<Q>(op + 192 * NR, od);
    E0 = e + o;
    E1 = e - o;
  } else if (wave == NCW) {
    // gradients and J1.  Shakhov relaxation and J1 of a value: -nu f + E c(xi)
    // with a cubic c per node and distribution (see the column shape)
    const double idx12 = P.inv_dx * (1.0 / 12.0);
    const int w = lane, j = w - 2;
    if (!j1) {
      if (j >= 0 && j < W)
        for (int m = 0; m < 4; ++m) S.co[MC_F + m][j] = S.co[MC_G + m][j] = 0.0;
    } else if (j >= 0 && j < W) {
      const double T = S.T[w], iT = rcpn(T);
      const double Ag = (S.X[w - 2] - 8.0 * S.X[w - 1] + 8.0 * S.X[w + 1] - S.X[w + 2]) * idx12 * rcpn(S.X[w]);
      const double Bg = (S.T[w - 2] - 8.0 * S.T[w - 1] + 8.0 * S.T[w + 1] - S.T[w + 2]) * idx12 * iT;
      const double Ug = (S.u[w - 2] - 8.0 * S.u[w - 1] + 8.0 * S.u[w + 1] - S.u[w + 2]) * idx12;
      const double pre = -P.b * nn * chi * cc;
      const double pA = pre * Ag, pB = pre * Bg, pU = pre * Ug;
      S.co[MC_F][j] = -0.6 * pU;
      S.co[MC_F + 1][j] = pA - 0.9 * pB;
      S.co[MC_F + 2][j] = 0.6 * pU * iT;
      S.co[MC_F + 3][j] = 0.3 * pB * iT;
      S.co[MC_G][j] = -0.2 * T * pU;
      S.co[MC_G + 1][j] = T * (pA - 0.3 * pB);
      S.co[MC_G + 2][j] = 0.6 * pU;
      S.co[MC_G + 3][j] = 0.3 * pB;
    }
  } else if (wave == NCW + 1) {
    if (lane < W) {
      double Fx = S.fp[0][lane];
#pragma unroll
      for (int q = 1; q < 64 / W; ++q) Fx += S.fp[q][lane];
      S.co[MC_FX][lane] = frc ? cc * (P.g_ext + Fx) : 0.0;
      S.co[MC_U][lane] = j0 || j1 ? S.u[lane + 2] : 0.0;
    }
  } else if (wave == NCW + 2) {
    // transport: mu (eq:viscosity), tau (eq:tau), Pr (eq:prandtl); J0
    if (!j0) {
      if (lane < W) {
        S.co[MC_NUB][lane] = bb;
        for (int m = 4; m < 7; ++m) S.co[MC_F + m][lane] = S.co[MC_G + m][lane] = 0.0;
      }
    } else if (lane < W) {
      const double T = S.T[lane + 2], n = S.n[lane + hn], chi = S.chi[lane + 2];
      const double bn = P.b * n;
      const double y = bn * chi;
      const double c12 = 0.16 * (1.0 + 12.0 / M_PI);
      const double c32 = 0.36 * (1.0 + 32.0 / (9.0 * M_PI));
      const double mu0 = P.mu0c * sqrt(T);
      const double mu = mu0 * (rcpn(chi) + 0.8 * bn + c12 * bn * bn * chi);
      const double Pr = (2.0 / 3.0) * (1.0 + 0.6 * y) * (1.0 + 0.8 * y + c12 * y * y) *
                        rcpn((1.0 + 0.4 * y) * (1.0 + 1.2 * y + c32 * y * y));
      const double iT = rcpn(T);
      const double nu = cc * chi * n * T * (1.0 + 0.4 * y) * rcpn(mu);
      const double sv = nu * ((1.0 - Pr) * qv * (0.2 * iT * iT) * rcpn(n));
      S.co[MC_NUB][lane] = bb - nu;
      S.co[MC_F + 4][lane] = nu;
      S.co[MC_F + 5][lane] = -3.0 * sv;
      S.co[MC_F + 6][lane] = sv * iT;
      S.co[MC_G + 4][lane] = T * nu;
      S.co[MC_G + 5][lane] = -T * sv;
      S.co[MC_G + 6][lane] = sv;
    }
  }
  __syncthreads();

  // ---- update ---------------------------------------------------------------
  if (wave < NCW) {
    const double* co = &S.co[d == 0 ? MC_F : MC_G][c];
    const double u = S.co[MC_U][c], nub = S.co[MC_NUB][c], fx = S.co[MC_FX][c];
    const double x0 = pr - u, x1 = -pr - u;
    acc0 = fma(nub, f0, fma(-fx, g0, acc0));
    acc1 = fma(nub, f1, fma(-fx, g1, acc1));
    const double k0 = co[0] + co[4 * W], k1 = co[W] + co[5 * W], k2 = co[2 * W], k3 = co[3 * W] + co[6 * W];
    const double o0 = fma(E0, fma(fma(fma(k3, x0, k2), x0, k1), x0, k0), acc0);
    const double o1 = fma(E1, fma(fma(fma(k3, x1, k2), x1, k1), x1, k0), acc1);
    if (valid) {
      A.f_out[(long long)row0 * ntot + gnode] = o0;
      A.f_out[(long long)row1 * ntot + gnode] = o1;
    }
    if (!A.rhs_mode) {
      const double m = mirror_blocks<Q>(mfma4(op[256 * NR + 64], o1, mfma4(op[256 * NR], o0, 0.0)));
      S.mom[d][lane >> 4][c] = m;
    }
  }
  if (A.rhs_mode) {
    __syncthreads();  // LDS is reused by the next tile
    return;
  }
  __syncthreads();

  // ---- moments of the new state ----------------------------------------------
  if (tid < W && i0 + tid < nsys) {
    const long long g = off + i0 + tid;
    const double n = S.mom[0][0][tid], m1 = S.mom[0][1][tid], m2 = S.mom[0][2][tid], m3 = S.mom[0][3][tid];
    const double e0 = S.mom[1][0][tid], e1 = S.mom[1][1][tid];
    const double in = rcpn(n);
    const double u = m1 * in;
    const double T = (2.0 / 3.0) * (0.5 * m2 + e0 - 0.5 * n * u * u) * in;
    const double x3 = m3 - 3.0 * u * m2 + 3.0 * u * u * m1 - u * u * u * n;
    const double q = 0.5 * x3 + e1 - u * e0;
    A.mom_out[g] = n;
    A.mom_out[ntot + g] = u;
    A.mom_out[2 * ntot + g] = tiso > 0.0 ? tiso : T;
    A.mom_out[3 * ntot + g] = q;
    if (!(n > 0.0) || !(T > 0.0) || !isfinite(n) || !isfinite(T) || !isfinite(q) || !isfinite(u))
      P.status[0] = 1;
  }
  __syncthreads();
}

// Workgroups go to the eight XCDs in turn (workgroup b to XCD b mod 8), and
// each XCD has its own L2.  xcd_tile gives XCD x the contiguous tiles
// x q + min(x, r) + i (ntiles = 8 q + r), so that tiles sharing halo and
// window lines, and a tile's own lines from one stage to the next, meet in
// one L2.  It is a bijection of 0 .. ntiles - 1.
__device__ __forceinline__ int xcd_tile(int b, int ntiles) {
  const int q = ntiles >> 3, r = ntiles & 7;
  const int x = b & 7, i = b >> 3;
  return x * q + min(x, r) + i;
}

// A grid of at most one workgroup per CU of an XCD runs on one alone: eight
// times as many are launched and those not on the first end at once.  The
// halos and moments that a stage reads then lie in the L2 that the previous
// stage wrote; from another XCD's they come over the memory side, a third of
// the load phase.  A stage of 256 nodes in a captured graph, spread over the
// XCDs -> on one: q 8 3.68 -> 3.42, q 16 3.91 -> 3.58, q 24 4.53 -> 4.23 us;
// with two workgroups per CU (1024 nodes, q 16) 3.91 -> 4.65.  The adjoint's
// kernels, longer chains of which the loads are a smaller part, gain nothing.
// Several contexts on streams of their own share that XCD and still gain: at
// most four hardware queues run at once, so a CU holds four workgroups at most.
// A stage of every context, captured, spread -> on one, us:
//   512 nodes   q 8   1 context 3.62 -> 3.38   2 4.00 -> 3.58   4 4.44 -> 3.67   8  8.84 ->  7.33
//               q 16            3.86 -> 3.61     4.30 -> 3.76     4.83 -> 3.92      9.44 ->  7.72
//               q 24            4.44 -> 4.39     4.79 -> 4.55     9.52 -> 9.00     14.77 -> 13.46
//   64 nodes    q 16            3.91 -> 3.58     4.10 -> 3.72     8.15 -> 7.41      8.83 ->  7.47
// Index of the workgroup in the grid, negative: not one of the grid's.
__device__ __forceinline__ int grid_index(const DevParams& P) {
  const int b = blockIdx.x;
  return P.onex ? (b & 7 ? -1 : b >> 3) : b;
}

// The leading arguments are what the first loads need: the build has the
// compiler ask for them in scalar registers at a wavefront's start (kernel
// argument preload, up to 14 dwords), so that these loads leave before the
// rest of the arguments, 400 bytes in memory, have come.  A stage of 256 nodes
// launched call by call: q 8 3.67 -> 3.47, q 16 3.77 -> 3.60, q 24 4.40 -> 4.22
// us (without the preload, 0.17 us slower than before).  tiles: null for a
// single system; 32 bits hold the node count of any state that fits.
template <int Q, int W, int TERMS>
__global__ __launch_bounds__((Mirror<Q, W>::NT)) void stage_kernel_mirror(const double* f_prev, const double* mom_in,
                                                                           const int4* tiles, const double* mx,
                                                                           int ntot, int hn, int ntiles, int onex,
                                                                           DevParams P, StageArgs A) {
  __shared__ SmemM<Q, W> S;
  A.f_prev = f_prev;
  A.mom_in = mom_in;
  P.tiles = tiles;
  P.mx = mx;
  P.ntot = ntot;
  P.hn = hn;
  P.ntiles = ntiles;
  P.single = tiles == nullptr;
  P.onex = onex;
  // one tile per workgroup (the grid is the tile count)
  const int b = grid_index(P);
  if (b >= 0 && b < P.ntiles) stage_tile_mirror<Q, W, TERMS>(P, A, P.onex ? b : xcd_tile(b, P.ntiles), S);
}

template <int Q, int W, int NG>
__global__ __launch_bounds__(W * NG) void stage_kernel(DevParams P, StageArgs A) {
  __shared__ Smem<Q, W, NG> S;
  load_tables<Q, W, NG>(P, S);
  if ((int)blockIdx.x < P.ntiles) stage_tile<Q, W, NG>(P, A, xcd_tile(blockIdx.x, P.ntiles), S);
}

// ---------------------------------------------------------------------------
// Column shape: one wavefront per tile of WC = 63 nodes, thread = node.  Each
// thread keeps its node's F, G columns (as sums and differences over mirror
// pairs of velocities) and Hermite moments in registers, so the contractions
// (equilibrium, momentum derivative) need no LDS traffic and the velocity
// moments of the new state are a per-thread sum.  The 64 lanes compute the 64
// WENO-5 faces of a row (face j between nodes j-1 and j); a node's right face
// comes from the next lane.
//
// An iteration forms the four values of a mirror pair (p_k, p_(Q-1-k)) of F and
// G: both contractions split into even and odd halves, half the multiplies
// and half the coefficients through the scalar cache, whose latency hides
// behind two faces each.  Bound by vector issue at two wavefronts per SIMD
// (the columns fill the registers, the tile a fifth or less of the LDS) and by
// the latency of the state's loads, which no other wavefront covers at small
// grids.  Requesting f_n an iteration ahead changed nothing.  A stage of 1.18 M
// nodes, value by value with full contractions -> by mirror pairs:
//   q 16  270 -> 224 us (3.6 TB/s of algorithmic bytes, 4.0 of traffic)   q 24  511 -> 348 us
// ---------------------------------------------------------------------------
constexpr int WC = 63;

// The density window is dead once the contact values and the forces are
// formed, and u, T and X of nodes -2..64 take its place: the tile then fits
// eight workgroups per CU (Q = 16).
template <int Q>
struct SmemCol {
  double f[2 * Q][WC + 2 * HF];      // columns: node i0 - 3 + c, c = 0..68
  union {
    double n[WC + 2 * HN_MAX];
    struct {
      double u[WC + 4], T[WC + 4], X[WC + 4];
    } g;
  } w;
  double sav[2 * MS_MAX + 1];        // averaging weights
  double cf[MF_MAX];                 // EV1 force taps
};

template <int Q, int TERMS>
__device__ void stage_tile_col(const DevParams& P, const StageArgs& A, int tile, SmemCol<Q>& S,
                               const double* __restrict__ vel, const double* __restrict__ pairs) {
  const int lane = threadIdx.x;  // 0..63
  const int4 td = P.tiles[tile];
  const int off = td.x, nsys = td.y, i0 = td.z;
  const long long ntot = P.ntot;
  const int hn = P.hn;
  const bool valid = lane < WC && (i0 + lane) < nsys;
  const long long gnode = off + i0 + lane;

  // ---- 1. load: own column to registers and LDS, halo columns to LDS ----
  double Fc[Q], Gc[Q];
  {
    const long long gown = off + wrapi(i0 + lane, nsys);  // lane 63: right halo node 63
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      Fc[k] = A.f_prev[(long long)k * ntot + gown];
      Gc[k] = A.f_prev[(long long)(Q + k) * ntot + gown];
    }
    // halo columns 0, 1, 2 (nodes -3..-1) and 67, 68 (nodes 64, 65) of all
    // 2Q rows, spread over the lanes: a few loads per lane instead of 2Q on
    // five lanes
    constexpr int NH = 5 * 2 * Q, LH = (NH + 63) / 64;
    double hv[LH];
#pragma unroll
    for (int i = 0; i < LH; ++i) {
      const int idx = lane + 64 * i;
      hv[i] = 0.0;
      if (idx < NH) {
        const int r = idx / 5, h = idx - 5 * r;
        const int c = h < 3 ? h : h + 64;
        hv[i] = A.f_prev[(long long)r * ntot + off + wrapi(i0 - HF + c, nsys)];
      }
    }
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      S.f[k][lane + HF] = Fc[k];
      S.f[Q + k][lane + HF] = Gc[k];
    }
#pragma unroll
    for (int i = 0; i < LH; ++i) {
      const int idx = lane + 64 * i;
      if (idx < NH) {
        const int r = idx / 5, h = idx - 5 * r;
        S.f[r][h < 3 ? h : h + 64] = hv[i];
      }
    }
  }
  // density window, u and T on nodes -2..64, the averaging and force tables:
  // all loads issued before the first LDS write
  const double* mn = A.mom_in;
  constexpr int LN = (WC + 2 * HN_MAX + 63) / 64;
  constexpr int LU = (WC + 4 + 63) / 64;
  static_assert(LU == 2, "nodes -2..64 on one or two values per lane");
  constexpr int NSAV = 2 * MS_MAX + 1;
  constexpr int LT = (NSAV + MF_MAX + 63) / 64;
  const int nwin = WC + 2 * hn;
  double nv[LN], uv[LU], Tv[LU], tv[LT];
#pragma unroll
  for (int i = 0; i < LN; ++i) {
    const int c = lane + 64 * i;
    nv[i] = c < nwin ? mn[off + wrapi(i0 - hn + c, nsys)] : 0.0;
  }
#pragma unroll
  for (int i = 0; i < LU; ++i) {
    const int c = lane + 64 * i;
    uv[i] = 0.0;
    Tv[i] = 0.0;
    if (c < WC + 4) {
      const int node = off + wrapi(i0 - 2 + c, nsys);
      uv[i] = mn[ntot + node];
      Tv[i] = mn[2 * ntot + node];
    }
  }
#pragma unroll
  for (int i = 0; i < LT; ++i) {
    const int e = lane + 64 * i;
    const double* src = nullptr;
    int si = 0;
    if (e < 2 * P.ms + 1) { src = P.savg; si = e; }
    else if (e >= NSAV && e < NSAV + P.mf) { src = P.cfor; si = e - NSAV; }
    tv[i] = src ? src[si] : 0.0;
  }
  const double qj = valid ? mn[3 * ntot + gnode] : 0.0;
  const double tiso = P.tiso && valid ? P.tiso[gnode] : P.T_iso;
#pragma unroll
  for (int i = 0; i < LN; ++i) {
    const int c = lane + 64 * i;
    if (c < nwin) S.w.n[c] = nv[i];
  }
#pragma unroll
  for (int i = 0; i < LT; ++i) {
    const int e = lane + 64 * i;
    if (e < NSAV) S.sav[e] = tv[i];
    else if (e < NSAV + MF_MAX) S.cf[e - NSAV] = tv[i];
  }
  __syncthreads();

  // ---- 2. contact value and X = n^2 chi T on nodes -2..64 (c = lane, and
  // c = lane + 64 on lanes 0..2), kept in registers ------------------------
  double chv[LU], Xv[LU];
#pragma unroll
  for (int i = 0; i < LU; ++i) {
    const int cc = lane + 64 * i;
    chv[i] = 1.0;
    Xv[i] = 1.0;
    if (cc < WC + 4) {
      // the averaging weights are even: pairs
      const double* nc = &S.w.n[cc + hn - 2];
      const double* sw = &S.sav[P.ms];
      const double nn = nc[0];
      double s0 = sw[0] * nn, s1 = 0.0;
      int j = 1;
      for (; j + 3 <= P.ms; j += 4) {
        s0 += sw[j] * (nc[j] + nc[-j]);
        s1 += sw[j + 1] * (nc[j + 1] + nc[-j - 1]);
        s0 += sw[j + 2] * (nc[j + 2] + nc[-j - 2]);
        s1 += sw[j + 3] * (nc[j + 3] + nc[-j - 3]);
      }
      for (; j <= P.ms; ++j) s0 += sw[j] * (nc[j] + nc[-j]);
      const double eta = P.eta_c * (s0 + s1);
      const double om = 1.0 - eta;
      chv[i] = (2.0 - eta) * rcpn(2.0 * om * om * om);
      Xv[i] = nn * nn * chv[i] * Tv[i];
    }
  }

  // ---- 3. node fields of the own node -------------------------------------
  const int jw = lane < WC ? lane : WC - 1;  // lane 63 mirrors lane 62 (no node)
  const int c = jw + 2, cn = jw + hn;
  const double n = S.w.n[cn];
  const double idx12 = P.inv_dx * (1.0 / 12.0);
  double Fx = P.g_ext;
  if (P.force_model == EVLB_FORCE_EV1) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int m = 1;
    for (; m + 3 <= P.mf; m += 4) {
      s0 += S.cf[m - 1] * (S.w.n[cn + m] - S.w.n[cn - m]);
      s1 += S.cf[m] * (S.w.n[cn + m + 1] - S.w.n[cn - m - 1]);
      s2 += S.cf[m + 1] * (S.w.n[cn + m + 2] - S.w.n[cn - m - 2]);
      s3 += S.cf[m + 2] * (S.w.n[cn + m + 3] - S.w.n[cn - m - 3]);
    }
    for (; m <= P.mf; ++m) s0 += S.cf[m - 1] * (S.w.n[cn + m] - S.w.n[cn - m]);
    Fx += (s0 + s1) + (s2 + s3);
  } else if (P.force_model == EVLB_FORCE_EV2) {
    const double d1 = (S.w.n[cn - 2] - 8.0 * S.w.n[cn - 1] + 8.0 * S.w.n[cn + 1] - S.w.n[cn + 2]) * idx12;
    const double d3 = (-S.w.n[cn - 2] + 2.0 * S.w.n[cn - 1] - 2.0 * S.w.n[cn + 1] + S.w.n[cn + 2]) *
                      (0.5 * P.inv_dx * P.inv_dx * P.inv_dx);
    Fx += P.two_a * d1 + P.kappa * d3;
  }
  __syncthreads();  // the density window is dead: u, T and X take its place
#pragma unroll
  for (int i = 0; i < LU; ++i) {
    const int cc = lane + 64 * i;
    if (cc < WC + 4) {
      S.w.g.u[cc] = uv[i];
      S.w.g.T[cc] = Tv[i];
      S.w.g.X[cc] = Xv[i];
    }
  }
  // chi of the own node (c = jw + 2) from the lane that formed it
  const int csrc = c < 64 ? c : c - 64;
  const double chA = __shfl(chv[0], csrc), chB = __shfl(chv[LU - 1], csrc);
  const double chi = c < 64 ? chA : chB;
  __syncthreads();
  // without collision terms the moments in them are those of an empty node at
  // rest
  const bool j0 = term_on<TERMS>(P, EVLB_TERM_J0), j1 = term_on<TERMS>(P, EVLB_TERM_J1);
  const double u = j0 || j1 ? S.w.g.u[c] : 0.0, T = j0 || j1 ? S.w.g.T[c] : 1.0;
  const double invT = rcpn(T);
  const double* Xs = S.w.g.X;
  const double* Ts = S.w.g.T;
  const double* us = S.w.g.u;
  const double Ag = (Xs[c - 2] - 8.0 * Xs[c - 1] + 8.0 * Xs[c + 1] - Xs[c + 2]) * idx12 * rcpn(Xs[c]);
  const double Bg = (Ts[c - 2] - 8.0 * Ts[c - 1] + 8.0 * Ts[c + 1] - Ts[c + 2]) * idx12 * invT;
  const double Ug = (us[c - 2] - 8.0 * us[c - 1] + 8.0 * us[c + 1] - us[c + 2]) * idx12;
  const double bn = P.b * n;
  const double y = bn * chi;
  const double c12 = 0.16 * (1.0 + 12.0 / M_PI);
  const double c32 = 0.36 * (1.0 + 32.0 / (9.0 * M_PI));
  const double mu = P.mu0c * sqrt(T) * (rcpn(chi) + 0.8 * bn + c12 * bn * bn * chi);
  const double nu = chi * n * T * (1.0 + 0.4 * y) * rcpn(mu);
  const double Pr = (2.0 / 3.0) * (1.0 + 0.6 * y) * (1.0 + 0.8 * y + c12 * y * y) *
                    rcpn((1.0 + 0.4 * y) * (1.0 + 1.2 * y + c32 * y * y));
  const double sS = (1.0 - Pr) * qj * (0.2 * invT * invT) * rcpn(n);
  const double pre = -bn * chi;
  // Hermite moments a_0 = n, a_1 = n u, a_{l+1} = u a_l + l (T - 1) a_{l-1}
  double a[Q];
  a[0] = j0 || j1 ? n : 0.0;
  a[1] = a[0] * u;
#pragma unroll
  for (int l = 1; l < Q - 1; ++l) a[l + 1] = fma(u, a[l], (double)l * (T - 1.0) * a[l - 1]);
  // even and odd parts of the columns over mirror pairs, f_j +- f_(Q-1-j)
#pragma unroll
  for (int j = 0; j < Q / 2; ++j) {
    const double f0 = Fc[j], f1 = Fc[Q - 1 - j], g0 = Gc[j], g1 = Gc[Q - 1 - j];
    Fc[j] = f0 + f1;
    Fc[Q - 1 - j] = f0 - f1;
    Gc[j] = g0 + g1;
    Gc[Q - 1 - j] = g0 - g1;
  }

  // ---- 4. update, mirror pair by mirror pair ------------------------------
  // out = ca f_n + bb f + cc L(f)
  const double cc = A.rhs_mode ? 1.0 : A.beta * P.dt;
  const double ca = A.rhs_mode || A.first ? 0.0 : A.alpha;
  const double bb = A.rhs_mode ? 0.0 : (A.first ? A.alpha + A.beta : A.beta);
  const bool base = !A.first && !A.rhs_mode && valid;
  const WenoK K = weno_k(P);
  const bool adv = term_on<TERMS>(P, EVLB_TERM_ADV), frc = term_on<TERMS>(P, EVLB_TERM_FORCE);
  // Shakhov relaxation and J1 of velocity k: -nu f_k + E_k c(xi) with
  // xi = p_k - u and a cubic c per node and distribution.  For F,
  //   nu (1 + sS xi (xi^2/T - 3)) + pre (xi (A + 0.3 (xi^2/T - 3) B) + 0.6 (xi^2/T - 1) U),
  // for G,
  //   nu T (1 + sS xi (xi^2/T - 1)) + pre T (xi (A + 0.3 (xi^2/T - 1) B) + 0.2 (3 xi^2/T - 1) U),
  // expanded in powers of xi and scaled by cc.
  const double nu0 = j0 ? cc * nu : 0.0, sv = j0 ? nu0 * sS : 0.0, pc = cc * pre;
  const double pA = j1 ? pc * Ag : 0.0, pB = j1 ? pc * Bg : 0.0, pU = j1 ? pc * Ug : 0.0;
  const double cF0 = nu0 - 0.6 * pU, cF1 = pA - 3.0 * sv - 0.9 * pB;
  const double cF2 = 0.6 * pU * invT, cF3 = (sv + 0.3 * pB) * invT;
  const double cG0 = T * (nu0 - 0.2 * pU), cG1 = T * (pA - sv - 0.3 * pB);
  const double cG2 = 0.6 * pU, cG3 = sv + 0.3 * pB;
  const double nub = bb - nu0, fx = cc * Fx, cdx = cc * P.inv_dx;
  double pm[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll 1
  for (int k = 0; k < Q / 2; ++k) {
    // rows r = 0: F_k, 1: F_(Q-1-k), 2: G_k, 3: G_(Q-1-k); p_k < 0
    const int kr[4] = {k, Q - 1 - k, Q + k, 2 * Q - 1 - k};
    double fb[4] = {0, 0, 0, 0};
    if (base) {
#pragma unroll
      for (int r = 0; r < 4; ++r) fb[r] = A.f_n[(long long)kr[r] * ntot + gnode];
    }
    // face `lane`, between nodes lane - 1 and lane, upwind by the sign of p:
    // columns lane + 1 .. lane + 5 from the right, lane .. lane + 4 from the left
    double v[4][5];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int m = 0; m < 5; ++m) v[r][m] = S.f[kr[r]][lane + m + (r & 1 ? 0 : 1)];
    const double own[4] = {v[0][2], v[1][3], v[2][2], v[3][3]};
    // face less the one on the right, the next lane's (lane 63's is not used)
    double d[4] = {0, 0, 0, 0};
    auto face = [&](int r) {
      const double h = r & 1 ? weno5(v[r][0], v[r][1], v[r][2], v[r][3], v[r][4], K)
                             : weno5(v[r][4], v[r][3], v[r][2], v[r][1], v[r][0], K);
      d[r] = h - wave_next(h);
    };
    // Scalar and LDS loads share a wait counter and scalar loads come back in
    // any order, so a wait for one is a wait for all: the LDS reads first, then
    // each half of the pair's coefficients goes out before two faces and is
    // used behind them (32 scalar registers at a time).
    asm volatile("" ::"v"(v[3][4]), "v"(v[2][4]), "v"(v[1][4]), "v"(v[0][4]));
    __builtin_amdgcn_sched_barrier(0);
    const double pk = vel[k];
    const double* row = pairs + k * 2 * Q;
    double dp[4] = {0, 0, 0, 0};
    double cd[Q];
    if (frc) {
#pragma unroll
      for (int j = 0; j < Q; ++j) cd[j] = row[Q + j];
    }
    __builtin_amdgcn_sched_barrier(0);
    if (adv) {
      face(0);
      face(1);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (frc) {
      // Dp f = odd +- even over mirror pairs
      double fe = 0.0, fo = 0.0, ge = 0.0, go = 0.0;
#pragma unroll
      for (int j = 0; j < Q / 2; ++j) {
        fe = fma(cd[j], Fc[j], fe);
        fo = fma(cd[Q / 2 + j], Fc[Q - 1 - j], fo);
        ge = fma(cd[j], Gc[j], ge);
        go = fma(cd[Q / 2 + j], Gc[Q - 1 - j], go);
      }
      dp[0] = fo + fe;
      dp[1] = fo - fe;
      dp[2] = go + ge;
      dp[3] = go - ge;
    }
    __builtin_amdgcn_sched_barrier(0);
    double ce[Q];
#pragma unroll
    for (int j = 0; j < Q; ++j) ce[j] = row[j];
    __builtin_amdgcn_sched_barrier(0);
    if (adv) {
      face(2);
      face(3);
    }
    __builtin_amdgcn_sched_barrier(0);
    // E = even + odd over the Hermite moments
    double ev = 0.0, od = 0.0;
#pragma unroll
    for (int j = 0; j < Q / 2; ++j) {
      ev = fma(ce[j], a[2 * j], ev);
      od = fma(ce[Q / 2 + j], a[2 * j + 1], od);
    }
    const double E[2] = {ev + od, ev - od};
    const double cx = cdx * pk, x0 = pk - u, x1 = -pk - u;
    const double q[4] = {fma(fma(fma(cF3, x0, cF2), x0, cF1), x0, cF0), fma(fma(fma(cF3, x1, cF2), x1, cF1), x1, cF0),
                         fma(fma(fma(cG3, x0, cG2), x0, cG1), x0, cG0), fma(fma(fma(cG3, x1, cG2), x1, cG1), x1, cG0)};
    double o[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      // the other terms of cc L(f) first, the states last: two roundings of the
      // size of the result, and that of nub
      double t = fma(-fx, dp[r], (r & 1 ? -cx : cx) * d[r]);
      t = fma(E[r & 1], q[r], t);
      o[r] = fma(ca, fb[r], fma(nub, own[r], t));
    }
    if (valid) {
#pragma unroll
      for (int r = 0; r < 4; ++r) A.f_out[(long long)kr[r] * ntot + gnode] = o[r];
    }
    const double sF = o[0] + o[1], tF = o[0] - o[1], sG = o[2] + o[3], tG = o[2] - o[3];
    const double p2 = pk * pk;
    pm[0] += sF;
    pm[1] = fma(pk, tF, pm[1]);
    pm[2] = fma(p2, sF, pm[2]);
    pm[3] = fma(p2 * pk, tF, pm[3]);
    pm[4] += sG;
    pm[5] = fma(pk, tG, pm[5]);
  }

  // ---- 5. moments of the new state ----------------------------------------
  if (!A.rhs_mode && valid) {
    const double n1 = pm[0];
    const double in1 = rcpn(n1);
    const double u1 = pm[1] * in1;
    const double T1 = (2.0 / 3.0) * (0.5 * pm[2] + pm[4] - 0.5 * n1 * u1 * u1) * in1;
    const double x3 = pm[3] - 3.0 * u1 * pm[2] + 3.0 * u1 * u1 * pm[1] - u1 * u1 * u1 * n1;
    const double q1 = 0.5 * x3 + pm[5] - u1 * pm[4];
    A.mom_out[gnode] = n1;
    A.mom_out[ntot + gnode] = u1;
    A.mom_out[2 * ntot + gnode] = tiso > 0.0 ? tiso : T1;
    A.mom_out[3 * ntot + gnode] = q1;
    if (!(n1 > 0.0) || !(T1 > 0.0) || !isfinite(n1) || !isfinite(T1) || !isfinite(q1) || !isfinite(u1))
      P.status[0] = 1;
  }
  __syncthreads();
}

template <int Q, int TERMS>
__global__ __launch_bounds__(64) void stage_kernel_col(DevParams P, StageArgs A, const double* __restrict__ vel,
                                                       const double* __restrict__ pairs) {
  __shared__ SmemCol<Q> S;
  // one tile per workgroup (the grid is the tile count)
  if ((int)blockIdx.x < P.ntiles) stage_tile_col<Q, TERMS>(P, A, xcd_tile(blockIdx.x, P.ntiles), S, vel, pairs);
}

// Grid-wide barrier for the persistent kernel (all workgroups co-resident:
// cooperative launch).  A monotonically increasing arrival counter: barrier
// number e completes when the counter reaches (e + 1) * nblocks.  An
// agent-scope release fence before the arrival and an acquire fence after
// the wait make each stage's global writes, from every XCD, visible to all
// workgroups.  The wait is bounded: on time-out the abort latch is set and
// every workgroup leaves its step loop.
__device__ bool grid_barrier(const DevParams& P, unsigned nblocks, unsigned epoch) {
  __syncthreads();
  __shared__ int s_ok;
  if (threadIdx.x == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __hip_atomic_fetch_add(P.bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned target = (epoch + 1u) * nblocks;
    int ok = 1;
    long long spins = 0;
    while ((int)(__hip_atomic_load(P.bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) < 0) {
      __builtin_amdgcn_s_sleep(1);
      if ((++spins & 1023) == 0) {
        if (spins > (1ll << 24) ||
            __hip_atomic_load(P.status + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
          __hip_atomic_store(P.status + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          ok = 0;
          break;
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    s_ok = ok;
  }
  __syncthreads();
  return s_ok != 0;
}

// Resets the barrier counter and the abort latch (a kernel rather than a
// memset so that the sequence stays valid under stream capture).
__global__ void clear_barrier_kernel(DevParams P) {
  if (threadIdx.x == 0) {
    P.bar[0] = 0u;
    P.bar[1] = 0u;
    P.status[1] = 0;
  }
}

struct PersistArgs {
  double* f;            // f^n in/out
  double* f1;
  double* f2;
  double* momA;
  double* momB;         // momA holds the moments of f on entry
  int nsteps;
};

// Persistent kernel: all stages of nsteps steps in one cooperative launch,
// workgroups separated by grid barriers between stages.
template <int Q, int W, int NG>
struct GroupShape {
  static constexpr int NT = W * NG;
  typedef Smem<Q, W, NG> Shared;
  __device__ static void prologue(const DevParams& P, Shared& S) { load_tables<Q, W, NG>(P, S); }
  __device__ static void tile(const DevParams& P, const StageArgs& A, int t, Shared& S, const double*, const double*) {
    stage_tile<Q, W, NG>(P, A, t, S);
  }
};

template <int Q, int W, int TERMS>
struct MirrorShape {
  static constexpr int NT = Mirror<Q, W>::NT;
  typedef SmemM<Q, W> Shared;
  __device__ static void prologue(const DevParams&, Shared&) {}
  __device__ static void tile(const DevParams& P, const StageArgs& A, int t, Shared& S, const double*, const double*) {
    stage_tile_mirror<Q, W, TERMS>(P, A, t, S);
  }
};

template <int Q>
struct ColumnShape {
  static constexpr int NT = 64;
  typedef SmemCol<Q> Shared;
  __device__ static void prologue(const DevParams&, Shared&) {}
  __device__ static void tile(const DevParams& P, const StageArgs& A, int t, Shared& S,
                              const double* __restrict__ vel, const double* __restrict__ pairs) {
    stage_tile_col<Q, ANY_TERMS>(P, A, t, S, vel, pairs);
  }
};

template <class SHAPE>
__global__ __launch_bounds__(SHAPE::NT) void persistent_kernel(DevParams P, PersistArgs R,
                                                               const double* __restrict__ vel,
                                                               const double* __restrict__ pairs) {
  __shared__ typename SHAPE::Shared S;
  SHAPE::prologue(P, S);
  const double a_s[3] = {0.0, 0.75, 1.0 / 3.0};
  const double b_s[3] = {1.0, 0.25, 2.0 / 3.0};
  unsigned epoch = 0;
  for (int step = 0; step < R.nsteps; ++step) {
    for (int s = 0; s < 3; ++s) {
      StageArgs A;
      A.f_prev = s == 0 ? R.f : (s == 1 ? R.f1 : R.f2);
      A.f_n = R.f;
      A.f_out = s == 0 ? R.f1 : (s == 1 ? R.f2 : R.f);
      const int parity = (step * 3 + s) & 1;
      A.mom_in = parity ? R.momB : R.momA;
      A.mom_out = parity ? R.momA : R.momB;
      A.alpha = a_s[s];
      A.beta = b_s[s];
      A.first = s == 0;
      A.rhs_mode = 0;
      for (int b = blockIdx.x; b < P.ntiles; b += gridDim.x) SHAPE::tile(P, A, xcd_tile(b, P.ntiles), S, vel, pairs);
      if (!grid_barrier(P, gridDim.x, epoch++)) return;
    }
  }
}

// Moments of a state, one thread per node (also the entry moments of a step).
template <int Q>
__global__ __launch_bounds__(64) void moments_kernel(const double* __restrict__ f, const double* __restrict__ vel,
                                                     int ntot, int onex, DevParams P,
                                                      double* __restrict__ n_out, double* __restrict__ u_out,
                                                      double* __restrict__ T_out, double* __restrict__ q_out,
                                                      int stage_input) {
  P.onex = onex;
  P.ntot = ntot;
  const int b = grid_index(P);
  const long long i = (long long)b * 64 + threadIdx.x;
  if (b < 0 || i >= P.ntot) return;
  const long long nt = P.ntot;
  double F[Q], G[Q];
  double n = 0.0, m1 = 0.0;
#pragma unroll
  for (int k = 0; k < Q; ++k) {
    F[k] = f[k * nt + i];
    G[k] = f[(Q + k) * nt + i];
    n += F[k];
    m1 += vel[k] * F[k];
  }
  const double u = m1 / n;
  double e = 0.0, q = 0.0;
#pragma unroll
  for (int k = 0; k < Q; ++k) {
    const double xi = vel[k] - u;
    const double ek = 0.5 * xi * xi * F[k] + G[k];
    e += ek;
    q += xi * ek;
  }
  const double T = (2.0 / 3.0) * e / n;
  n_out[i] = n;
  u_out[i] = u;
  // as the input of a stage, an isothermal run sees its fixed temperature
  const double tiso = stage_input ? (P.tiso ? P.tiso[i] : P.T_iso) : 0.0;
  T_out[i] = tiso > 0.0 ? tiso : T;
  if (q_out) q_out[i] = q;
}

// Reduced Maxwellian F = E(n, u, T), G = T E, one thread per node.
template <int Q>
__global__ __launch_bounds__(256) void equilibrium_kernel(DevParams P, const double* __restrict__ n_in,
                                                          const double* __restrict__ u_in,
                                                          const double* __restrict__ T_in,
                                                          double* __restrict__ f) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P.ntot) return;
  const long long nt = P.ntot;
  const double n = n_in[i], u = u_in[i], T = T_in[i];
  double a[Q];
  a[0] = n;
  a[1] = n * u;
#pragma unroll
  for (int l = 1; l < Q - 1; ++l) a[l + 1] = u * a[l] + (double)l * (T - 1.0) * a[l - 1];
#pragma unroll
  for (int k = 0; k < Q; ++k) {
    double E = 0.0;
#pragma unroll
    for (int l = 0; l < Q; ++l) E += P.meq[k * Q + l] * a[l];
    f[k * nt + i] = E;
    f[(Q + k) * nt + i] = T * E;
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

#include "adjoint.inc"

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

constexpr int WIDE = 64;    // tile width for large grids
constexpr int NARROW = WN;  // tile width for grids too small to fill the chip

constexpr int WB = 32;    // nodes per broad mirror tile (q 8 and 16)
constexpr int BROAD = 1;  // launch shape code: broad mirror tiles

struct Layout {
  size_t tables, mx, tiles_broad, tiles_wide, tiles_narrow, tiles_col, tiles_adj, f1, f2, momA, momB, status, tiso;
  size_t adj_g, adj_mu2, adj_mu1, adj_fa, adj_mom, adj_part, adj_lam, total;
  long long ntot;
  size_t mirror;  // bytes of the mirror shapes' tables and broad tiles
  int ntiles_broad, ntiles_wide, ntiles_narrow, ntiles_col, ntiles_adj, ms, mf;
  size_t ntables;
};

int count_tiles(const evlb_params* p, int w) {
  int t = 0;
  for (int s = 0; s < p->n_sys; ++s) t += (p->nx[s] + w - 1) / w;
  return t;
}

bool is_even_multiple(double a, double dx, int* m, double tol = 1e-9) {
  const double r = a / dx;
  const long long k = llround(r);
  if (k <= 0 || std::fabs(r - (double)k) > tol * r || (k & 1)) return false;
  *m = (int)k;
  return true;
}

int validate(const evlb_params* p) {
  if (!p) return EVLB_EINVAL;
  if (p->abi_version != EVLB_ABI_VERSION) return EVLB_EINVAL;
  if (p->dim == 2) return p->T_iso_sys ? EVLB_EUNSUPPORTED : evlb2d::validate(p);
  if (p->dim != 1) return EVLB_EUNSUPPORTED;
  if (p->n_sys < 1 || !p->nx) return EVLB_EINVAL;
  long long ntot = 0;
  for (int s = 0; s < p->n_sys; ++s) {
    if (p->nx[s] < 8) return EVLB_EINVAL;
    ntot += p->nx[s];
  }
  if (ntot > (1ll << 31) - 1) return EVLB_EINVAL;
  if (p->q != 8 && p->q != 16 && p->q != 24) return EVLB_EUNSUPPORTED;
  if (!(p->dx > 0) || !(p->dt > 0) || !std::isfinite(p->dx) || !std::isfinite(p->dt)) return EVLB_EINVAL;
  if (!(p->sigma > 0) || !(p->phi_sigma >= 0) || !std::isfinite(p->phi_sigma)) return EVLB_EINVAL;
  if (!(p->gamma > 3.0)) return EVLB_EINVAL;
  if (p->force_model == EVLB_FORCE_EV2 && !(p->gamma > 5.0)) return EVLB_EINVAL;
  if (p->force_model < 0 || p->force_model > 2) return EVLB_EINVAL;
  if (p->term_mask & ~EVLB_TERM_ALL) return EVLB_EINVAL;
  if (!(p->weno_eps > 0) || !std::isfinite(p->g_ext)) return EVLB_EINVAL;
  if (p->exec_mode < 0 || p->exec_mode > 2) return EVLB_EINVAL;
  if (p->adjoint != 0 && p->adjoint != 1) return EVLB_EINVAL;
  if (p->adjoint && p->force_model == EVLB_FORCE_EV2) return EVLB_EUNSUPPORTED;
  if (!(p->T_iso >= 0.0) || !std::isfinite(p->T_iso)) return EVLB_EINVAL;
  if (p->adjoint && p->T_iso > 0.0) return EVLB_EUNSUPPORTED;
  if (p->T_iso_sys) {
    for (int s = 0; s < p->n_sys; ++s) {
      const double t = p->T_iso_sys[s];
      if (!(t >= 0.0) || !std::isfinite(t)) return EVLB_EINVAL;
      if (p->adjoint && t > 0.0) return EVLB_EUNSUPPORTED;
    }
  }
  if (p->tile_nodes != 0 && p->tile_nodes != WIDE && p->tile_nodes != NARROW && p->tile_nodes != WC)
    return EVLB_EINVAL;
  int ms, mf = 0;
  // the averaging window is the nearest even number of cells; sigma may sit
  // slightly off it (derivatives with respect to sigma at a fixed window)
  if (!is_even_multiple(p->sigma, p->dx, &ms, 1e-3) || ms > MS_MAX) return EVLB_EINVAL;
  if (p->force_model == EVLB_FORCE_EV1) {
    if (!is_even_multiple(p->r_cut, p->dx, &mf) || mf > MF_MAX) return EVLB_EINVAL;
  }
  // stability of WENO-5 + TVD-RK3 advection: CFL number <= 1
  std::vector<double> v, w;
  evlb::gauss_hermite_nodes(p->q, v, w);
  if (p->dt * v.back() / p->dx > 1.0) return EVLB_ECFL;
  return EVLB_OK;
}

// MFMA operands per lane of the mirror shape, and their values: lane L of
// operand i at 64 i + L, in the order Dp even, Dp odd, meq even, meq odd (one
// for each block that holds parts of r, by distance), then p_r^i and p_(q-1-r)^i.
int mirror_operands(int q) { return q == 8 ? Mirror<8, WN>::NOP : (q == 16 ? Mirror<16, WN>::NOP : Mirror<24, WN>::NOP); }

std::vector<double> mirror_table(int q, const evlb::HostTables& t) {
  const int KT = q / 8, NR = (mirror_operands(q) - 2) / 4;
  auto part = [&](int b) { return q == 8 ? 0 : (q == 16 ? b >> 1 : b); };  // kt of a block
  std::vector<double> x((size_t)64 * (4 * NR + 2), 0.0);
  for (int L = 0; L < 64; ++L) {
    const int i = L & 3, b = (L >> 2) & 3, k = L >> 4;
    if (part(b) >= KT) continue;
    const int row = KT * i + part(b);
    for (int s = 0; s < NR; ++s) {
      const int src = part((b - (q == 16 ? 2 * s : s)) & 3);
      if (src >= KT) continue;
      const int j = KT * k + src;
      const double dj = t.dpm[(size_t)row * q + j], dm = t.dpm[(size_t)row * q + q - 1 - j];
      x[64 * s + L] = 0.5 * (dj + dm);
      x[64 * (NR + s) + L] = 0.5 * (dj - dm);
      x[64 * (2 * NR + s) + L] = t.meq[(size_t)row * q + 2 * j];
      x[64 * (3 * NR + s) + L] = t.meq[(size_t)row * q + 2 * j + 1];
    }
    const double p = t.vel[KT * k + part(b)], m = i == 0 ? 1.0 : (i == 1 ? p : (i == 2 ? p * p : p * p * p));
    x[64 * (4 * NR) + L] = m;
    x[64 * (4 * NR + 1) + L] = i & 1 ? -m : m;
  }
  return x;
}

// Coefficients of the mirror pair (p_k, p_(q-1-k)), k < q / 2: meq[k] over the
// even, then the odd Hermite moments; (Dp[k][j] + Dp[k][q-1-j]) / 2, then their
// difference's half, j < q / 2.  (Dp f)_k and (Dp f)_(q-1-k) are odd +- even of
// these over f_j -+ f_(q-1-j), for Dp[q-1-k][q-1-j] = -Dp[k][j].
std::vector<double> pair_table(int q, const evlb::HostTables& t) {
  std::vector<double> x;
  for (int k = 0; k < q / 2; ++k) {
    for (int o = 0; o < 2; ++o)
      for (int j = 0; j < q / 2; ++j) x.push_back(t.meq[(size_t)k * q + 2 * j + o]);
    for (int o = 0; o < 2; ++o)
      for (int j = 0; j < q / 2; ++j) {
        const double d0 = t.dpm[(size_t)k * q + j], d1 = t.dpm[(size_t)k * q + q - 1 - j];
        x.push_back(0.5 * (o == 0 ? d0 + d1 : d0 - d1));
      }
  }
  return x;
}

Layout make_layout(const evlb_params* p) {
  Layout L{};
  L.ntot = 0;
  for (int s = 0; s < p->n_sys; ++s) L.ntot += p->nx[s];
  L.ntiles_broad = count_tiles(p, WB);
  L.ntiles_wide = count_tiles(p, WIDE);
  L.ntiles_narrow = count_tiles(p, NARROW);
  L.ntiles_col = count_tiles(p, WC);
  L.ntiles_adj = count_tiles(p, WA);
  L.ms = (int)llround(p->sigma / p->dx);
  L.mf = p->force_model == EVLB_FORCE_EV1 ? (int)llround(p->r_cut / p->dx) : 0;
  const int q = p->q;
  size_t off = 0;
  L.tables = off;
  const int mfa = L.mf > 0 ? L.mf : 1;
  L.ntables = (size_t)(q + 2 * q * q + 2 * (2 * L.ms + 1) + 3 * mfa);
  off += align256(sizeof(double) * L.ntables);
  L.mx = off;
  off += align256(sizeof(double) * (64 * (size_t)mirror_operands(q) + NTAB + (size_t)q * q));
  L.tiles_broad = off;
  off += align256(sizeof(int4) * (size_t)L.ntiles_broad);
  L.mirror = off - L.mx;
  L.tiles_wide = off;
  off += align256(sizeof(int4) * (size_t)L.ntiles_wide);
  L.tiles_narrow = off;
  off += align256(sizeof(int4) * (size_t)L.ntiles_narrow);
  L.tiles_col = off;
  off += align256(sizeof(int4) * (size_t)L.ntiles_col);
  L.tiles_adj = off;
  off += align256(sizeof(int4) * (size_t)L.ntiles_adj);
  const size_t fbytes = align256(sizeof(double) * 2 * (size_t)q * (size_t)L.ntot);
  L.f1 = off; off += fbytes;
  L.f2 = off; off += fbytes;
  const size_t mbytes = align256(sizeof(double) * 4 * (size_t)L.ntot);
  L.momA = off; off += mbytes;
  L.momB = off; off += mbytes;
  L.status = off; off += 256;
  L.tiso = 0;
  if (p->T_iso_sys) {
    L.tiso = off;
    off += align256(sizeof(double) * (size_t)L.ntot);
  }
  if (p->adjoint) {
    L.adj_g = off; off += fbytes;
    L.adj_mu2 = off; off += fbytes;
    L.adj_mu1 = off; off += fbytes;
    L.adj_fa = off; off += align256(sizeof(double) * NFA * (size_t)L.ntot);
    L.adj_mom = off; off += mbytes;
    // parameter partials: per VJP one slot per field-adjoint tile (16 nodes) and per node tile, for two
    // steps (a step's partials are summed while the next step runs)
    L.adj_part = off; off += align256(sizeof(double) * 2 * 2 * 3 * (size_t)(L.ntiles_narrow + L.ntiles_adj));
    L.adj_lam = off; off += fbytes;
  }
  L.total = off;
  return L;
}

}  // namespace

struct evlb_ctx {
  evlb_params p;
  std::vector<int32_t> nx;
  std::vector<double> vel;
  std::vector<double> tiso;  // per-system isothermal temperatures (copy of T_iso_sys)
  Layout L;
  DevParams dp;  // tiles/ntiles of the wide shape; launches patch them
  char* ws;
  int device;
  int cus;
  evlb2d::Ctx* c2 = nullptr;  // dim = 2 path
};

namespace {

#define EVLB_HIP(call)                         \
  do {                                         \
    if ((call) != hipSuccess) return EVLB_EHIP; \
  } while (0)

// launch shapes per quadrature order: wide tiles of 64 nodes, NG groups
template <int Q> struct WideNG;
template <> struct WideNG<8> { static constexpr int v = 4; };
template <> struct WideNG<16> { static constexpr int v = 8; };
template <> struct WideNG<24> { static constexpr int v = 8; };

// whether the narrow tiles, at one per CU, fit one XCD (see grid_index)
bool one_xcd(const evlb_ctx* c) { return 8 * c->L.ntiles_narrow <= c->cus; }

// workgroups to launch for a grid of n
unsigned grid_of(const DevParams& P, int n) { return P.onex ? 8u * (unsigned)(n - 1) + 1u : (unsigned)n; }

DevParams params_for(const evlb_ctx* c, int w) {
  DevParams P = c->dp;
  if (w == NARROW) {
    P.tiles = (const int4*)(c->ws + c->L.tiles_narrow);
    P.ntiles = c->L.ntiles_narrow;
    P.onex = one_xcd(c);
  } else if (w == BROAD) {
    P.tiles = (const int4*)(c->ws + c->L.tiles_broad);
    P.ntiles = c->L.ntiles_broad;
  } else if (w == WC) {
    P.tiles = (const int4*)(c->ws + c->L.tiles_col);
    P.ntiles = c->L.ntiles_col;
  } else {
    P.tiles = (const int4*)(c->ws + c->L.tiles_wide);
    P.ntiles = c->L.ntiles_wide;
  }
  return P;
}

template <int Q, int W, int NG>
int launch_stage(evlb_ctx* c, const StageArgs& A, hipStream_t st) {
  const DevParams P = params_for(c, W);
  hipLaunchKernelGGL((stage_kernel<Q, W, NG>), dim3(P.ntiles), dim3(W * NG), 0, st, P, A);
  return hipGetLastError() == hipSuccess ? EVLB_OK : EVLB_EHIP;
}

template <int Q, int W>
int launch_stage_mirror(evlb_ctx* c, const StageArgs& A, hipStream_t st) {
  const DevParams P = params_for(c, W == NARROW ? NARROW : BROAD);
  // The branches on the mask lie in the node wavefronts' chains: with all terms
  // known a stage of 256 nodes (q 16) takes 3.38, by the mask 3.47 us.
  const auto kernel = P.term_mask == EVLB_TERM_ALL ? stage_kernel_mirror<Q, W, EVLB_TERM_ALL>
                                                   : stage_kernel_mirror<Q, W, ANY_TERMS>;
  hipLaunchKernelGGL(kernel, dim3(grid_of(P, P.ntiles)), dim3(Mirror<Q, W>::NT), 0, st, A.f_prev, A.mom_in,
                     P.single ? nullptr : P.tiles, P.mx, (int)P.ntot, P.hn, P.ntiles, P.onex, P, A);
  return hipGetLastError() == hipSuccess ? EVLB_OK : EVLB_EHIP;
}

template <int Q>
int launch_stage_col(evlb_ctx* c, const StageArgs& A, hipStream_t st) {
  const DevParams P = params_for(c, WC);
  // The faces and the momentum derivative known to be in or out: behind runtime
  // conditions they spill up to 142 scalar registers in the loop over the pairs.
  // A right-hand side of the force alone, q 24: 25000 nodes 25.8 -> 18.5, 40000
  // 33.8 -> 23.1, 64000 38.5 -> 27.5 us.
  const int af = P.term_mask & (EVLB_TERM_ADV | EVLB_TERM_FORCE);
  const auto kernel = P.term_mask == EVLB_TERM_ALL ? stage_kernel_col<Q, EVLB_TERM_ALL>
                      : af == 0                    ? stage_kernel_col<Q, 0>
                      : af == EVLB_TERM_ADV        ? stage_kernel_col<Q, EVLB_TERM_ADV>
                      : af == EVLB_TERM_FORCE      ? stage_kernel_col<Q, EVLB_TERM_FORCE>
                                                   : stage_kernel_col<Q, EVLB_TERM_ADV | EVLB_TERM_FORCE>;
  hipLaunchKernelGGL(kernel, dim3(P.ntiles), dim3(64), 0, st, P, A, P.vel, P.pairs);
  return hipGetLastError() == hipSuccess ? EVLB_OK : EVLB_EHIP;
}

template <class SHAPE>
int launch_persistent(evlb_ctx* c, int width, double* f, int nsteps, hipStream_t st) {
  int per_cu = 0;
  EVLB_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, persistent_kernel<SHAPE>, SHAPE::NT, 0));
  if (per_cu < 1) return EVLB_EHIP;
  // every workgroup waits for all others at the grid barrier: only as many as
  // are sure to be resident (a workgroup takes further tiles in turn)
  constexpr int waves = SHAPE::NT / 64;
  if (evlb::uneven(waves)) {
    hipFuncAttributes attr;
    EVLB_HIP(hipFuncGetAttributes(&attr, (const void*)persistent_kernel<SHAPE>));
    per_cu = evlb::resident_per_cu(per_cu, waves, attr.numRegs);
  }
  DevParams P = params_for(c, width);
  int grid = per_cu * c->cus;
  if (grid > P.ntiles) grid = P.ntiles;
  PersistArgs R;
  R.f = f;
  R.f1 = (double*)(c->ws + c->L.f1);
  R.f2 = (double*)(c->ws + c->L.f2);
  R.momA = (double*)(c->ws + c->L.momA);
  R.momB = (double*)(c->ws + c->L.momB);
  R.nsteps = nsteps;
  hipLaunchKernelGGL(clear_barrier_kernel, dim3(1), dim3(64), 0, st, P);
  EVLB_HIP(hipGetLastError());
  const double* vel = P.vel;
  const double* pairs = P.pairs;
  void* args[] = {&P, &R, &vel, &pairs};
  EVLB_HIP(hipLaunchCooperativeKernel((const void*)persistent_kernel<SHAPE>, dim3(grid), dim3(SHAPE::NT), args, 0, st));
  return EVLB_OK;
}

template <int Q>
int run_moments(evlb_ctx* c, const double* f, double* n, double* u, double* T, double* q, hipStream_t st,
                int stage_input = 1) {
  const long long nt = c->L.ntot;
  DevParams P = c->dp;
  P.onex = one_xcd(c);
  hipLaunchKernelGGL((moments_kernel<Q>), dim3(grid_of(P, (int)((nt + 63) / 64))), dim3(64), 0, st, f, P.vel,
                     (int)nt, P.onex, P, n, u, T, q, stage_input);
  return hipGetLastError() == hipSuccess ? EVLB_OK : EVLB_EHIP;
}

// Tile shape of the per-stage launches: explicit, or by the number of tiles.
// A stage in us on 256 CUs, narrow / broad / column:
//   q 8    4096 nodes 4.7 / 5.0 / 8.8   5120 5.2 / 4.8 / 8.8   40960 15 / 10.3 / 10.8   49152 17 / 11.7 / 11.0
//   q 16   4096 nodes 5.0 / 5.6 / 12    5120 5.7 / 5.5 / 12    40960 18 / 15.8 / 15.5   49152 21 / 18.3 / 16.6
//   q 24   4096 nodes 5.7 / - / 17      8192 7.5 / - / 17      24576 18.3 / - / 18.8    32768 23.6 / - / 20.1
// Narrow tiles while they fill the CUs once: the stage is one tile's latency,
// and a broad one's is longer.  Beyond that broad tiles for q 8 and 16, which
// hold fewer halos and node fields formed twice (q 24 would need two
// workgroups' lanes).  The column shape, one wavefront a tile with the fewest
// instructions per value, from two and a half tiles per CU on, for q 24 one
// and a half.  The tile of 64 nodes is not in the rule.  It is ahead of what the
// rule takes only about where that changes to the column shape, captured, rule /
// 64: q 24 16384 nodes 11.5 / 11.2, 24576 17.8 / 16.3, 32768 19.1 / 17.6, 40960
// 19.8 / 23.6; q 16 40960 14.3 / 17.3; q 8 65536 13.1 / 12.8.
int pick_width(const evlb_ctx* c) {
  if (c->p.tile_nodes) return c->p.tile_nodes;
  if (2 * c->L.ntiles_col > (c->p.q < 24 ? 5 : 3) * c->cus) return WC;
  return c->p.q < 24 && c->L.ntiles_narrow > c->cus ? BROAD : NARROW;
}

// of the persistent launch, whose grid barrier waits for every workgroup: the
// broad shape is not built for it
int pick_width_persistent(const evlb_ctx* c) {
  if (c->p.tile_nodes) return c->p.tile_nodes;
  return c->L.ntiles_col >= 4 * c->cus ? WC : NARROW;
}

StageArgs stage_args(double* f, double* f1, double* f2, double* momA, double* momB, int step, int s) {
  const double a_s[3] = {0.0, 0.75, 1.0 / 3.0};
  const double b_s[3] = {1.0, 0.25, 2.0 / 3.0};
  StageArgs A;
  A.f_prev = s == 0 ? f : (s == 1 ? f1 : f2);
  A.f_n = f;
  A.f_out = s == 0 ? f1 : (s == 1 ? f2 : f);
  const int parity = (step * 3 + s) & 1;
  A.mom_in = parity ? momB : momA;
  A.mom_out = parity ? momA : momB;
  A.alpha = a_s[s];
  A.beta = b_s[s];
  A.first = s == 0;
  A.rhs_mode = 0;
  return A;
}

template <int Q>
int launch_stage_w(evlb_ctx* c, int w, const StageArgs& A, hipStream_t st) {
  if (w == NARROW) return launch_stage_mirror<Q, NARROW>(c, A, st);
  if (w == WC) return launch_stage_col<Q>(c, A, st);
  if constexpr (Q < 24) {
    if (w == BROAD) return launch_stage_mirror<Q, WB>(c, A, st);
  }
  return launch_stage<Q, WIDE, WideNG<Q>::v>(c, A, st);
}

template <int Q>
int run_step(evlb_ctx* c, double* f, int nsteps, hipStream_t st) {
  const long long nt = c->L.ntot;
  double* momA = (double*)(c->ws + c->L.momA);
  double* momB = (double*)(c->ws + c->L.momB);
  int rc = run_moments<Q>(c, f, momA, momA + nt, momA + 2 * nt, momA + 3 * nt, st);
  if (rc) return rc;
  int mode = c->p.exec_mode;
  if (mode == EVLB_EXEC_AUTO) mode = EVLB_EXEC_PER_STAGE;
  const int w = mode == EVLB_EXEC_PERSISTENT ? pick_width_persistent(c) : pick_width(c);
  if (mode == EVLB_EXEC_PERSISTENT) {
    if (w == NARROW)
      return c->p.term_mask == EVLB_TERM_ALL
                 ? launch_persistent<MirrorShape<Q, NARROW, EVLB_TERM_ALL>>(c, w, f, nsteps, st)
                 : launch_persistent<MirrorShape<Q, NARROW, ANY_TERMS>>(c, w, f, nsteps, st);
    if (w == WC) return launch_persistent<ColumnShape<Q>>(c, w, f, nsteps, st);
    return launch_persistent<GroupShape<Q, WIDE, WideNG<Q>::v>>(c, w, f, nsteps, st);
  }
  double* f1 = (double*)(c->ws + c->L.f1);
  double* f2 = (double*)(c->ws + c->L.f2);
  for (int step = 0; step < nsteps; ++step) {
    for (int s = 0; s < 3; ++s) {
      rc = launch_stage_w<Q>(c, w, stage_args(f, f1, f2, momA, momB, step, s), st);
      if (rc) return rc;
    }
  }
  return EVLB_OK;
}

template <int Q>
int run_rhs(evlb_ctx* c, const double* f, double* L, hipStream_t st) {
  const long long nt = c->L.ntot;
  double* momA = (double*)(c->ws + c->L.momA);
  double* momB = (double*)(c->ws + c->L.momB);
  int rc = run_moments<Q>(c, f, momA, momA + nt, momA + 2 * nt, momA + 3 * nt, st);
  if (rc) return rc;
  StageArgs A;
  A.f_prev = f;
  A.f_n = f;
  A.f_out = L;
  A.mom_in = momA;
  A.mom_out = momB;
  A.alpha = 0.0;
  A.beta = 1.0;
  A.first = 1;
  A.rhs_mode = 1;
  return launch_stage_w<Q>(c, pick_width(c), A, st);
}

template <int Q>
int run_equilibrium(evlb_ctx* c, const double* n, const double* u, const double* T, double* f, hipStream_t st) {
  const int blocks = (int)((c->L.ntot + 255) / 256);
  hipLaunchKernelGGL((equilibrium_kernel<Q>), dim3(blocks), dim3(256), 0, st, c->dp, n, u, T, f);
  return hipGetLastError() == hipSuccess ? EVLB_OK : EVLB_EHIP;
}


// ---- adjoint step -----------------------------------------------------------

DevParams params_adj(const evlb_ctx* c) {
  DevParams P = c->dp;
  P.tiles = (const int4*)(c->ws + c->L.tiles_adj);
  P.ntiles = c->L.ntiles_adj;
  return P;
}

// g = (dL/df)^T v at state f (moments mom), written as
// out = cc (v + dt g) + a1 X1 + a2 X2; parameter partials weighted by pw into
// the slot range vjp_index of the partial buffer (one slot per field-adjoint
// tile, then one per node tile).
template <int Q>
int launch_vjp(evlb_ctx* c, const double* f, const double* mom, const double* v, double* out, const double* X1,
               const double* X2, double cc, double a1, double a2, double pw, int vjp_index, hipStream_t st,
               double* vinj = nullptr, const double* obs = nullptr, const double* wts = nullptr, int j = 0,
               bool final_reduce = false, double* dparams = nullptr, int par = 0, bool sum_prev = false) {
  const DevParams P = params_adj(c);
  AdjArgs A;
  A.f = f;
  A.mom = mom;
  A.v = v;
  A.gdir = (double*)(c->ws + c->L.adj_g);
  A.fa = (double*)(c->ws + c->L.adj_fa);
  A.out = out;
  A.X1 = X1;
  A.X2 = X2;
  A.c = cc;
  A.a1 = a1;
  A.a2 = a2;
  A.pw = pw;
  A.vinj = vinj;
  A.obs = obs;
  A.w = wts;
  A.j = j;
  const int nta = P.ntiles;
  const DevParams Pn = params_for(c, NARROW);
  const int ntn = Pn.ntiles;
  const int nslots = 3 * (ntn + nta);  // one step: three VJPs
  // slots of step parity par, VJP i: ntn field-adjoint tiles, then nta node tiles
  double* part = (double*)(c->ws + c->L.adj_part) + (size_t)par * 2 * nslots;
  // with sum_prev, one extra field workgroup sums the other parity's slots
  // (the previous step, complete by stream order) into dparams
  A.rpart = sum_prev ? (const double*)(c->ws + c->L.adj_part) + (size_t)(par ^ 1) * 2 * nslots : nullptr;
  A.rslots = nslots;
  A.rdp = dparams;
  A.part = part + (size_t)vjp_index * 2 * (ntn + nta);
  hipLaunchKernelGGL((adj_fields_kernel<Q>), dim3(ntn + (sum_prev ? 1 : 0)), dim3(WN * Q + 256), 0, st, A.f, A.mom, A.v,
                     Pn.single ? nullptr : Pn.tiles, (int)Pn.ntot, Pn.hn, ntn, Pn, A);
  EVLB_HIP(hipGetLastError());
  A.rpart = nullptr;
  A.part = part + ((size_t)vjp_index * (ntn + nta) + ntn) * 2;
  hipLaunchKernelGGL((adj_column_kernel<Q>), dim3(nta * (2 * Q / NCR)), dim3(64 * NCW), 0, st, A.f, A.mom, A.v, A.fa,
                     P.single ? nullptr : P.tiles, (int)P.ntot, nta, P.ms,
                     P.force_model == EVLB_FORCE_EV1 ? P.mf : 0, P, A, final_reduce ? 1 : 0, (const double*)part,
                     nslots, dparams);
  EVLB_HIP(hipGetLastError());
  return EVLB_OK;
}

// One adjoint step given the step's states f^n, f1, f2 and their moments.
template <int Q>
int adjoint_core(evlb_ctx* c, const double* fn, const double* mn, const double* f1, const double* m1,
                 const double* f2, const double* m2, const double* lam3, double* lam0, double* dparams,
                 hipStream_t st, double* lam3_inject = nullptr, const double* obs = nullptr,
                 const double* wts = nullptr, int j = 0, int par = 0, bool sum_prev = false,
                 bool final_reduce = true) {
  double* mu2 = (double*)(c->ws + c->L.adj_mu2);
  double* mu1 = (double*)(c->ws + c->L.adj_mu1);
  const double dt = c->p.dt;
  // f^{n+1} = 1/3 f^n + 2/3 (f2 + dt L(f2)):   mu2 = 2/3 (lam3 + dt J(f2)^T lam3)
  // (with an observable: lam3 += w[j] obs first, stored back into lam3)
  // (with sum_prev, the previous step's parameter partials are summed into
  // dparams beside the first kernel)
  int rc = launch_vjp<Q>(c, f2, m2, lam3, mu2, nullptr, nullptr, 2.0 / 3.0, 0.0, 0.0, dt * 2.0 / 3.0, 0, st,
                         lam3_inject, obs, wts, j, false, dparams, par, sum_prev);
  if (rc) return rc;
  // f2 = 3/4 f^n + 1/4 (f1 + dt L(f1)):          mu1 = 1/4 (mu2 + dt J(f1)^T mu2)
  rc = launch_vjp<Q>(c, f1, m1, mu2, mu1, nullptr, nullptr, 0.25, 0.0, 0.0, dt * 0.25, 1, st, nullptr, nullptr,
                     nullptr, 0, false, nullptr, par);
  if (rc) return rc;
  // f1 = f^n + dt L(f^n):  lam^n = mu1 + dt J(f^n)^T mu1 + 1/3 lam3 + 3/4 mu2
  // (with final_reduce its last kernel adds the step's parameter derivatives
  // to dparams; otherwise the next step's first kernel does)
  return launch_vjp<Q>(c, fn, mn, mu1, lam0, lam3, mu2, 1.0, 1.0 / 3.0, 0.75, dt, 2, st, nullptr, nullptr, nullptr, 0,
                       final_reduce, dparams, par);
}

template <int Q>
int run_adjoint(evlb_ctx* c, const double* fn, const double* lam3, double* lam0, double* dparams, hipStream_t st) {
  const long long nt = c->L.ntot;
  double* momA = (double*)(c->ws + c->L.momA);
  double* momB = (double*)(c->ws + c->L.momB);
  double* f1 = (double*)(c->ws + c->L.f1);
  double* f2 = (double*)(c->ws + c->L.f2);
  double* amom = (double*)(c->ws + c->L.adj_mom);
  // recompute the two inner stages: f1 (moments in momB), f2 (moments in momA)
  int rc = run_moments<Q>(c, fn, amom, amom + nt, amom + 2 * nt, amom + 3 * nt, st);
  if (rc) return rc;
  const int w = pick_width(c);
  StageArgs A0 = stage_args(const_cast<double*>(fn), f1, f2, momA, momB, 0, 0);
  A0.mom_in = amom;
  rc = launch_stage_w<Q>(c, w, A0, st);
  if (rc) return rc;
  rc = launch_stage_w<Q>(c, w, stage_args(const_cast<double*>(fn), f1, f2, momA, momB, 0, 1), st);
  if (rc) return rc;
  return adjoint_core<Q>(c, fn, amom, f1, momB, f2, momA, lam3, lam0, dparams, st);
}

// Record layout of one step j: f^j, f1^j, f2^j ([2][q][n] each), then the
// moments of the three ([4][n] each).
size_t record_doubles(const evlb_ctx* c) {
  const size_t fs = 2 * (size_t)c->p.q * (size_t)c->L.ntot;
  return 3 * fs + 3 * 4 * (size_t)c->L.ntot;
}

template <int Q>
int run_step_record(evlb_ctx* c, const double* f0, int nsteps, double* rec, hipStream_t st) {
  const size_t fs = 2 * (size_t)Q * (size_t)c->L.ntot;
  const size_t R = record_doubles(c);
  const long long nt = c->L.ntot;
  EVLB_HIP(hipMemcpyAsync(rec, f0, fs * sizeof(double), hipMemcpyDeviceToDevice, st));
  double* m0 = rec + 3 * fs;
  int rc = run_moments<Q>(c, rec, m0, m0 + nt, m0 + 2 * nt, m0 + 3 * nt, st);
  if (rc) return rc;
  const int w = pick_width(c);
  const double a_s[3] = {0.0, 0.75, 1.0 / 3.0};
  const double b_s[3] = {1.0, 0.25, 2.0 / 3.0};
  for (int j = 0; j < nsteps; ++j) {
    double* r = rec + (size_t)j * R;
    double* rn = rec + (size_t)(j + 1) * R;
    double* fj[3] = {r, r + fs, r + 2 * fs};
    double* mj[3] = {r + 3 * fs, r + 3 * fs + 4 * nt, r + 3 * fs + 8 * nt};
    for (int s = 0; s < 3; ++s) {
      StageArgs A;
      A.f_prev = fj[s];
      A.f_n = fj[0];
      A.f_out = s < 2 ? fj[s + 1] : rn;
      A.mom_in = mj[s];
      A.mom_out = s < 2 ? mj[s + 1] : rn + 3 * fs;
      A.alpha = a_s[s];
      A.beta = b_s[s];
      A.first = s == 0;
      A.rhs_mode = 0;
      rc = launch_stage_w<Q>(c, w, A, st);
      if (rc) return rc;
    }
  }
  return EVLB_OK;
}

template <int Q>
int run_adjoint_record(evlb_ctx* c, const double* rec, int nsteps, double* lam, const double* obs, const double* wts,
                       double* dparams, hipStream_t st) {
  const size_t fs = 2 * (size_t)Q * (size_t)c->L.ntot;
  const size_t R = record_doubles(c);
  const long long nt = c->L.ntot;
  double* other = (double*)(c->ws + c->L.adj_lam);
  double* cur = lam;
  for (int j = nsteps - 1; j >= 0; --j) {
    const double* r = rec + (size_t)j * R;
    double* nxt = cur == lam ? other : lam;
    const bool inj = obs && wts;
    // step s of the pass keeps its parameter partials in parity s & 1; the
    // next step sums them beside its first kernel, and the last step sums its
    // own in its last kernel
    const int s = nsteps - 1 - j;
    int rc = adjoint_core<Q>(c, r, r + 3 * fs, r + fs, r + 3 * fs + 4 * nt, r + 2 * fs, r + 3 * fs + 8 * nt, cur, nxt,
                             dparams, st, inj ? cur : nullptr, obs, wts, j, s & 1, s > 0, j == 0);
    if (rc) return rc;
    cur = nxt;
  }
  if (cur != lam) EVLB_HIP(hipMemcpyAsync(lam, cur, fs * sizeof(double), hipMemcpyDeviceToDevice, st));
  return EVLB_OK;
}

template <int Q>
int run_equilibrium_adjoint(evlb_ctx* c, const double* n, const double* u, const double* T, const double* lam,
                            double* nb, double* ub, double* Tb, hipStream_t st) {
  const int blocks = (int)((c->L.ntot + 255) / 256);
  hipLaunchKernelGGL((equilibrium_adjoint_kernel<Q>), dim3(blocks), dim3(256), 0, st, c->dp, n, u, T, lam, nb, ub,
                     Tb);
  return hipGetLastError() == hipSuccess ? EVLB_OK : EVLB_EHIP;
}

#define EVLB_DISPATCH_Q(q, fn, ...)              \
  switch (q) {                                   \
    case 8: return fn<8>(__VA_ARGS__);           \
    case 16: return fn<16>(__VA_ARGS__);         \
    case 24: return fn<24>(__VA_ARGS__);         \
    default: return EVLB_EUNSUPPORTED;           \
  }

bool device_matches(const evlb_ctx* c) {
  int d = -1;
  return hipGetDevice(&d) == hipSuccess && d == c->device;
}

}  // namespace

// The workspace of evlb_init_noalloc: one array per device, loaded with the
// code object.  Host code reaches it only through the address that
// hipGetSymbolAddress returns with that device current (the array's name in
// host code is a host-side stand-in, not a device address).
// The limit does not count the mirror shapes' tables and broad tiles, for which
// it has NOALLOC_TABLES more: 15 KiB and 16 bytes per broad tile (in systems of
// the 8 nodes that a system has at least, and q 8, one per 2.5 KiB).
constexpr size_t NOALLOC_TABLES = (size_t)512 << 10;
static __device__ __align__(256) unsigned char scratch[EVLB_NOALLOC_MAX_BYTES + NOALLOC_TABLES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch[kMaxDevices];  // device address of `scratch` per device (null: not looked up yet)

int scratch_address(int device, void** out) {
  if (device < 0 || device >= kMaxDevices) return EVLB_EHIP;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[device]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return EVLB_EHIP;
    g_scratch[device] = p;
  }
  *out = g_scratch[device];
  return EVLB_OK;
}
}  // namespace

extern "C" {

int evlb_validate(const evlb_params* params) { return validate(params); }

size_t evlb_workspace_bytes(const evlb_params* params) {
  if (validate(params) != EVLB_OK) return 0;
  if (params->dim == 2) return evlb2d::workspace_bytes(params);
  return make_layout(params).total;
}

int evlb_init_noalloc(const evlb_params* params, void* hip_stream, evlb_ctx** out) {
  if (!out) return EVLB_EINVAL;
  *out = nullptr;
  const int rc = validate(params);
  if (rc) return rc;
  const size_t need = evlb_workspace_bytes(params);
  const size_t tables = params->dim == 2 ? 0 : make_layout(params).mirror;
  if (need - tables > EVLB_NOALLOC_MAX_BYTES || need > sizeof(scratch)) return EVLB_EWORKSPACE;
  int device = -1;
  if (hipGetDevice(&device) != hipSuccess) return EVLB_EHIP;
  void* ws = nullptr;
  const int sc = scratch_address(device, &ws);
  if (sc) return sc;
  return evlb_init(params, ws, sizeof(scratch), hip_stream, out);
}

int evlb_init(const evlb_params* params, void* d_workspace, size_t ws_bytes, void* hip_stream, evlb_ctx** out) {
  if (!out) return EVLB_EINVAL;
  *out = nullptr;
  int rc = validate(params);
  if (rc) return rc;
  if (params->dim == 2) {
    const size_t need = evlb2d::workspace_bytes(params);
    if (!d_workspace || ws_bytes < need || ((uintptr_t)d_workspace & 255)) return EVLB_EWORKSPACE;
    evlb_ctx* c = new (std::nothrow) evlb_ctx();
    if (!c) return EVLB_EINVAL;
    c->p = *params;
    c->nx.assign(params->nx, params->nx + 1);
    c->p.nx = c->nx.data();
    if (hipGetDevice(&c->device) != hipSuccess) { delete c; return EVLB_EHIP; }
    rc = evlb2d::init(params, (char*)d_workspace, ws_bytes, (hipStream_t)hip_stream, &c->c2);
    if (rc) { delete c; return rc; }
    c->ws = (char*)d_workspace;
    c->vel = evlb2d::velocities(c->c2);
    c->L.ntot = evlb2d::node_count(c->c2);
    c->dp.status = evlb2d::status_word(c->c2);
    *out = c;
    return EVLB_OK;
  }
  const Layout L = make_layout(params);
  if (!d_workspace || ws_bytes < L.total || ((uintptr_t)d_workspace & 255)) return EVLB_EWORKSPACE;
  evlb_ctx* c = new (std::nothrow) evlb_ctx();
  if (!c) return EVLB_EINVAL;
  c->p = *params;
  c->nx.assign(params->nx, params->nx + params->n_sys);
  c->p.nx = c->nx.data();
  if (params->T_iso_sys) c->tiso.assign(params->T_iso_sys, params->T_iso_sys + params->n_sys);
  c->p.T_iso_sys = params->T_iso_sys ? c->tiso.data() : nullptr;
  c->L = L;
  c->ws = (char*)d_workspace;
  if (hipGetDevice(&c->device) != hipSuccess) { delete c; return EVLB_EHIP; }
  if (hipDeviceGetAttribute(&c->cus, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess) {
    delete c;
    return EVLB_EHIP;
  }
  evlb::TableParams tp{params->q, params->dx, params->sigma, params->phi_sigma, params->gamma, params->r_cut};
  evlb::HostTables t;
  evlb::build_tables(tp, t);
  if (params->force_model != EVLB_FORCE_EV1) {
    t.cfor.assign(1, 0.0);
    t.cphi.assign(1, 0.0);
    t.csig.assign(1, 0.0);
  }
  c->vel = t.vel;
  const int q = params->q;
  std::vector<double> host;
  host.insert(host.end(), t.vel.begin(), t.vel.end());
  host.insert(host.end(), t.meq.begin(), t.meq.end());
  host.insert(host.end(), t.dpm.begin(), t.dpm.end());
  host.insert(host.end(), t.savg.begin(), t.savg.end());
  host.insert(host.end(), t.cfor.begin(), t.cfor.end());
  host.insert(host.end(), t.cphi.begin(), t.cphi.end());
  host.insert(host.end(), t.csig.begin(), t.csig.end());
  host.insert(host.end(), t.ssig.begin(), t.ssig.end());
  std::vector<double> mx = mirror_table(q, t);
  const size_t ntab = mx.size();
  mx.resize(ntab + NTAB, 0.0);
  const size_t npairs = mx.size();
  const std::vector<double> pairs = pair_table(q, t);
  mx.insert(mx.end(), pairs.begin(), pairs.end());
  std::copy(t.savg.begin(), t.savg.end(), mx.begin() + ntab);
  if (L.mf > 0) std::copy(t.cfor.begin(), t.cfor.end(), mx.begin() + ntab + TAB_CF);
  std::vector<int4> tb, tw, tn, tc, ta;
  int off = 0;
  for (int s = 0; s < params->n_sys; ++s) {
    for (int i0 = 0; i0 < params->nx[s]; i0 += WB) tb.push_back(make_int4(off, params->nx[s], i0, 0));
    for (int i0 = 0; i0 < params->nx[s]; i0 += WIDE) tw.push_back(make_int4(off, params->nx[s], i0, 0));
    for (int i0 = 0; i0 < params->nx[s]; i0 += NARROW) tn.push_back(make_int4(off, params->nx[s], i0, 0));
    for (int i0 = 0; i0 < params->nx[s]; i0 += WC) tc.push_back(make_int4(off, params->nx[s], i0, 0));
    for (int i0 = 0; i0 < params->nx[s]; i0 += WA) ta.push_back(make_int4(off, params->nx[s], i0, 0));
    off += params->nx[s];
  }
  hipStream_t st = (hipStream_t)hip_stream;
  double* tab = (double*)(c->ws + L.tables);
  // the per-system temperatures expanded to one value per node
  std::vector<double> tn_node;
  if (params->T_iso_sys) {
    tn_node.resize((size_t)L.ntot);
    size_t o = 0;
    for (int s = 0; s < params->n_sys; ++s)
      for (int i = 0; i < params->nx[s]; ++i) tn_node[o++] = params->T_iso_sys[s];
  }
  // copies ordered on the caller's stream; the stream is synchronised before
  // returning because the host vectors die with this call
  if (hipMemcpyAsync(c->ws + L.mx, mx.data(), mx.size() * sizeof(double), hipMemcpyHostToDevice, st) != hipSuccess ||
      hipMemcpyAsync(tab, host.data(), host.size() * sizeof(double), hipMemcpyHostToDevice, st) != hipSuccess ||
      hipMemcpyAsync(c->ws + L.tiles_broad, tb.data(), tb.size() * sizeof(int4), hipMemcpyHostToDevice, st) !=
          hipSuccess ||
      hipMemcpyAsync(c->ws + L.tiles_wide, tw.data(), tw.size() * sizeof(int4), hipMemcpyHostToDevice, st) !=
          hipSuccess ||
      hipMemcpyAsync(c->ws + L.tiles_narrow, tn.data(), tn.size() * sizeof(int4), hipMemcpyHostToDevice, st) !=
          hipSuccess ||
      hipMemcpyAsync(c->ws + L.tiles_col, tc.data(), tc.size() * sizeof(int4), hipMemcpyHostToDevice, st) !=
          hipSuccess ||
      hipMemcpyAsync(c->ws + L.tiles_adj, ta.data(), ta.size() * sizeof(int4), hipMemcpyHostToDevice, st) !=
          hipSuccess ||
      hipMemsetAsync(c->ws + L.status, 0, 256, st) != hipSuccess ||
      (params->T_iso_sys && hipMemcpyAsync(c->ws + L.tiso, tn_node.data(), tn_node.size() * sizeof(double),
                                           hipMemcpyHostToDevice, st) != hipSuccess) ||
      hipStreamSynchronize(st) != hipSuccess) {
    delete c;
    return EVLB_EHIP;
  }
  DevParams& d = c->dp;
  d.vel = tab;
  d.meq = tab + q;
  d.mx = (const double*)(c->ws + L.mx);
  d.ntab = d.mx + ntab;
  d.pairs = d.mx + npairs;
  d.dpm = tab + q + q * q;
  d.savg = tab + q + 2 * q * q;
  const int nc = (int)t.cfor.size();
  d.cfor = tab + q + 2 * q * q + 2 * L.ms + 1;
  d.cphi = d.cfor + nc;
  d.csig = d.cphi + nc;
  d.ssig = d.csig + nc;
  d.tiles = (const int4*)(c->ws + L.tiles_wide);
  d.ntiles = L.ntiles_wide;
  d.single = params->n_sys == 1;
  d.ms = L.ms;
  d.mf = L.mf;
  d.hn = L.mf > L.ms + 2 ? L.mf : L.ms + 2;
  d.ntot = L.ntot;
  d.dx = params->dx;
  d.inv_dx = 1.0 / params->dx;
  d.dt = params->dt;
  const double sg = params->sigma;
  d.b = 2.0 * M_PI * sg * sg * sg / 3.0;
  d.eta_c = M_PI * sg * sg * sg / 6.0;
  d.mu0c = 5.0 / (16.0 * sg * sg * std::sqrt(M_PI));
  d.sigma = sg;
  d.weno_eps = params->weno_eps;
  d.weno_e3 = 0.3 * params->weno_eps;
  d.weno_e75 = 0.75 * params->weno_eps;
  d.g_ext = params->g_ext;
  const double g = params->gamma;
  d.two_a = 2.0 * (2.0 * M_PI * sg * sg * sg / 3.0) * params->phi_sigma * g / (g - 3.0);
  d.kappa = (2.0 * M_PI * std::pow(sg, 5) / 15.0) * params->phi_sigma * (g > 5.0 ? g / (g - 5.0) : 0.0);
  d.force_model = params->force_model;
  d.term_mask = params->term_mask;
  d.T_iso = params->T_iso;
  d.tiso = params->T_iso_sys ? (const double*)(c->ws + L.tiso) : nullptr;
  d.status = (int*)(c->ws + L.status);
  d.bar = (unsigned*)(c->ws + L.status + 64);
  *out = c;
  return EVLB_OK;
}

int evlb_set_equilibrium(evlb_ctx* ctx, const double* d_n, const double* d_u, const double* d_T, double* d_f,
                         void* hip_stream) {
  if (!ctx || !d_n || !d_u || !d_T || !d_f) return EVLB_EINVAL;
  if (!device_matches(ctx)) return EVLB_EINVAL;
  if (ctx->c2) return evlb2d::set_equilibrium(ctx->c2, d_n, d_u, d_T, d_f, (hipStream_t)hip_stream);
  EVLB_DISPATCH_Q(ctx->p.q, run_equilibrium, ctx, d_n, d_u, d_T, d_f, (hipStream_t)hip_stream);
}

int evlb_step(evlb_ctx* ctx, double* d_f, int32_t nsteps, void* hip_stream) {
  if (!ctx || !d_f || nsteps < 0) return EVLB_EINVAL;
  if (!device_matches(ctx)) return EVLB_EINVAL;
  if (nsteps == 0) return EVLB_OK;
  if (ctx->c2) return evlb2d::step(ctx->c2, d_f, nsteps, (hipStream_t)hip_stream);
  EVLB_DISPATCH_Q(ctx->p.q, run_step, ctx, d_f, nsteps, (hipStream_t)hip_stream);
}

int evlb_rhs(evlb_ctx* ctx, const double* d_f, double* d_L, void* hip_stream) {
  if (!ctx || !d_f || !d_L || d_f == d_L) return EVLB_EINVAL;
  if (!device_matches(ctx)) return EVLB_EINVAL;
  if (ctx->c2) return evlb2d::rhs(ctx->c2, d_f, d_L, (hipStream_t)hip_stream);
  EVLB_DISPATCH_Q(ctx->p.q, run_rhs, ctx, d_f, d_L, (hipStream_t)hip_stream);
}

int evlb_moments(evlb_ctx* ctx, const double* d_f, double* d_n, double* d_u, double* d_T, double* d_q,
                 void* hip_stream) {
  if (!ctx || !d_f || !d_n || !d_u || !d_T) return EVLB_EINVAL;
  if (!device_matches(ctx)) return EVLB_EINVAL;
  if (ctx->c2) return evlb2d::moments(ctx->c2, d_f, d_n, d_u, d_T, d_q, (hipStream_t)hip_stream);
  EVLB_DISPATCH_Q(ctx->p.q, run_moments, ctx, d_f, d_n, d_u, d_T, d_q, (hipStream_t)hip_stream, 0);
}

int evlb_adjoint_step(evlb_ctx* ctx, const double* d_f_n, const double* d_lam_np1, double* d_lam_n,
                      double* d_dparams, void* hip_stream) {
  if (!ctx || !d_f_n || !d_lam_np1 || !d_lam_n || !d_dparams) return EVLB_EINVAL;
  if (ctx->c2) return EVLB_EUNSUPPORTED;
  if (!ctx->p.adjoint) return EVLB_EINVAL;
  if (d_lam_n == d_lam_np1 || (const double*)d_lam_n == d_f_n) return EVLB_EINVAL;
  if (!device_matches(ctx)) return EVLB_EINVAL;
  EVLB_DISPATCH_Q(ctx->p.q, run_adjoint, ctx, d_f_n, d_lam_np1, d_lam_n, d_dparams, (hipStream_t)hip_stream);
}

int evlb_equilibrium_adjoint(evlb_ctx* ctx, const double* d_n, const double* d_u, const double* d_T,
                             const double* d_lam, double* d_nbar, double* d_ubar, double* d_Tbar, void* hip_stream) {
  if (!ctx || !d_n || !d_u || !d_T || !d_lam || !d_nbar || !d_ubar || !d_Tbar) return EVLB_EINVAL;
  if (ctx->c2) return EVLB_EUNSUPPORTED;
  if (!device_matches(ctx)) return EVLB_EINVAL;
  EVLB_DISPATCH_Q(ctx->p.q, run_equilibrium_adjoint, ctx, d_n, d_u, d_T, d_lam, d_nbar, d_ubar, d_Tbar,
                  (hipStream_t)hip_stream);
}

int64_t evlb_record_doubles(const evlb_ctx* ctx) { return ctx && !ctx->c2 ? (int64_t)record_doubles(ctx) : 0; }

int evlb_step_record(evlb_ctx* ctx, const double* d_f0, int32_t nsteps, double* d_rec, void* hip_stream) {
  if (!ctx || !d_f0 || !d_rec || nsteps < 0) return EVLB_EINVAL;
  if (ctx->c2) return EVLB_EUNSUPPORTED;
  if (!device_matches(ctx)) return EVLB_EINVAL;
  EVLB_DISPATCH_Q(ctx->p.q, run_step_record, ctx, d_f0, nsteps, d_rec, (hipStream_t)hip_stream);
}

int evlb_adjoint_record(evlb_ctx* ctx, const double* d_rec, int32_t nsteps, double* d_lam, const double* d_obs,
                        const double* d_w, double* d_dparams, void* hip_stream) {
  if (!ctx || !d_rec || !d_lam || !d_dparams || nsteps < 0) return EVLB_EINVAL;
  if (ctx->c2) return EVLB_EUNSUPPORTED;
  if (!ctx->p.adjoint || ((d_obs == nullptr) != (d_w == nullptr))) return EVLB_EINVAL;
  if (!device_matches(ctx)) return EVLB_EINVAL;
  EVLB_DISPATCH_Q(ctx->p.q, run_adjoint_record, ctx, d_rec, nsteps, d_lam, d_obs, d_w, d_dparams,
                  (hipStream_t)hip_stream);
}

int evlb_status(evlb_ctx* ctx, void* hip_stream, int32_t clear) {
  if (!ctx) return EVLB_EINVAL;
  hipStream_t st = (hipStream_t)hip_stream;
  int h[2] = {0, 0};
  // read (and clear) the latch in stream order, then wait for both
  if (hipMemcpyAsync(h, ctx->dp.status, sizeof(h), hipMemcpyDeviceToHost, st) != hipSuccess) return EVLB_EHIP;
  if (clear && hipMemsetAsync(ctx->dp.status, 0, sizeof(h), st) != hipSuccess) return EVLB_EHIP;
  if (hipStreamSynchronize(st) != hipSuccess) return EVLB_EHIP;
  if (h[1]) return EVLB_EHIP;
  return h[0] ? EVLB_ENONFINITE : EVLB_OK;
}

int evlb_info(const evlb_ctx* ctx, int64_t* n_tot, double* h_velocities) {
  if (!ctx) return EVLB_EINVAL;
  if (n_tot) *n_tot = ctx->L.ntot;
  if (h_velocities) std::memcpy(h_velocities, ctx->vel.data(), ctx->vel.size() * sizeof(double));
  return EVLB_OK;
}

void evlb_destroy(evlb_ctx* ctx) {
  if (ctx && ctx->c2) evlb2d::destroy(ctx->c2);
  delete ctx;
}

const char* evlb_strerror(int code) {
  switch (code) {
    case EVLB_OK: return "ok";
    case EVLB_EINVAL: return "invalid argument or parameter";
    case EVLB_ECFL: return "time step above the advection stability limit";
    case EVLB_EWORKSPACE: return "workspace missing, too small or not 256-byte aligned";
    case EVLB_EHIP: return "HIP runtime error";
    case EVLB_ENONFINITE: return "non-positive or non-finite density or temperature";
    case EVLB_EUNSUPPORTED: return "unsupported configuration";
    default: return "unknown error";
  }
}

}  // extern "C"
