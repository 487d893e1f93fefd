// Workgroups that are resident on a CU together, for a launch whose workgroups
// wait for one another.  Host arithmetic only.
#pragma once

namespace evlb {

// whether a workgroup's wavefronts may lie unevenly on the four SIMDs
constexpr bool uneven(int wavefronts) { return wavefronts % 4 != 0 && wavefronts > 1; }

// The occupancy query counts a CU's wavefront slots in one sum.  A CU has four
// SIMDs, each with slots of its own, and deals a workgroup's wavefronts round
// them from where it stands: six wavefronts are 2 + 2 + 1 + 1, and two such
// workgroups need not become 3 + 3 + 3 + 3.  With three slots a SIMD (158
// registers a lane) the query says two of them fit, and a grid barrier over two
// per CU timed out.  Whole quads of wavefronts lie evenly, and a lone one takes
// any slot; otherwise each SIMD has to hold a workgroup's larger share.
// registers: vector registers a lane, of 512 in units of 8; at most 8 slots.
inline int resident_per_cu(int occupancy, int wavefronts, int registers) {
  if (!uneven(wavefronts)) return occupancy;
  const int units = registers > 8 ? (registers + 7) / 8 : 1;
  const int slots = 64 / units < 8 ? 64 / units : 8;
  const int fit = slots / ((wavefronts + 3) / 4);
  return fit < occupancy ? (fit > 0 ? fit : 1) : occupancy;
}

}  // namespace evlb
