// rules.hpp -- host rules of the dispatch that depend on sizes only: which
// kernel form or tile a level takes.  Every form gives the same bits.
#pragma once
#include <algorithm>
#include <cmath>

#include "geometry.hpp"

namespace lbm {

// k_fine3s (both D3Q19 BGK / RR fine substeps in one marching pass) addresses
// the storage window of its run (zlen + 4 planes and one storage block) and
// the compact x-band copy with 32-bit byte offsets, both below 2^31.  Longest
// run of planes it can take on this fine level; 0: none.
template <typename S>
inline int fine3_zcap(const Geo& g) {
  constexpr int Q = 19;
  if ((double)xband_elems(g, Q) * sizeof(S) >= 2147483648.0) return 0;
  const double plane = (double)g.pf * g.nf[1] * Q * sizeof(S);
  const double room = 2147483648.0 - 2.0 * (double)PopBlock<S>::B * Q * sizeof(S);
  return std::max(0, (int)std::floor(room / plane) - 4);
}

}  // namespace lbm
