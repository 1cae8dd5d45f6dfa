// rules.hpp -- host rules of the dispatch that depend on sizes only: which
// kernel form or tile a level takes.  Every form gives the same bits.
#pragma once
#include <algorithm>
#include <cmath>

#include "geometry.hpp"

namespace lbm {

// FP32 wide tiles of the marching D3Q19 kernels (variant 2): 130 x 7 lanes, or
// 194 x 5 where 192 columns a tile leave fewer idle than 128 in rows of n nodes
// (129 to 192, 513 to 576, 897 to 960 and so on).  Fine kernel with 130 x 7 / 194 x 5 /
// 66 x 15 lanes, us: RR 139^3 212 / 169 / 192, 159^3 277 / 229 / 246, 179^3 361 / 290 /
// 308, 199^3 (256 or 384 columns) 471 / 617 / 447; H-RR 139^3 169 / 123 / 153, 179^3
// 317 / 226 / 272, 199^3 407 / 532 / 381.  Step, us: 577 x 201 x 201 RR 1244 / 1198 /
// 1221, H-RR 2337 / 2225 / 2239; 521 x 161 x 161 RR 820 / 810 / 804, H-RR 1513 / 1471 /
// 1451; coarse H-RR 550 x 180 x 180 852 / 825 / 779, 576 x 180 x 180 804 / 817 / 721.
inline bool wide194(int n) { return (n + 191) / 192 * 192 < (n + 127) / 128 * 128; }

// FP32 fine levels whose middle rows of n nodes take 66 x 15 tiles (variant 3) by
// default.  Between 193 and 256 nodes 130 x 7 and 66 x 15 tiles leave the same
// columns idle; the shorter halo wins while these are many, us a step with
// 130 x 7 / 66 x 15: 193^3 H-RR 1039 / 980, 207^3 RR 625 / 601, H-RR 1203 / 1174;
// 223^3 RR 771 / 822, H-RR 1419 / 1483, 239^3 RR 884 / 947, H-RR 1623 / 1720.  Up to
// 128 nodes BGK / RR takes 66 x 15 (127^3 188 / 174; in rows of 95 to 119 nodes the
// other is up to 6 % ahead).
inline bool tall66(int n, bool hrr) { return (n > 192 && n < 216) || (n <= 128 && !hrr); }

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

// Default of the fine role of a D3Q19 BGK / RR level of `bytes` (two buffers):
// whether its substeps run as one marching kernel (k_fine3s) or as two
// launches.  One work group a CU needs some planes of tiles to fill the
// device: from 100 MB, in double (where small levels also share launches with
// the interface, Grid::kTail) from 500 MB.  us a step in two launches / in one:
// FP32 65^3 55 / 75, 97^3 119 / 111, 129^3 235 / 225; FP64 81^3 115 / 129, 97^3
// 182 / 194, 113^3 285 / 287, 129^3 399 / 379.
// Thin levels keep the two launches, which waste less on them: short rows
// leave columns of a tile idle, few rows or planes give short runs and idle
// CUs, and a level of 250 to 600 MB, which the memory-side cache half holds,
// loses least by its second pass.  Nodes of the level, us in two / in one:
// FP32 to 600 MB, rows of 72: 61 x 121 x 121 98 / 118, 67 x 201 x 201 291 / 313, 81 x
// 201 x 201 334 / 320.  To 170 MB, in rows of 129 on of 130 x 7 or 194 x 5 tiles, sides
// of 15: 181 x 181 x 29 99 / 91, 401 x 41 x 61 97 / 82, 401 x 121 x 17 90 / 86, 241 x 241 x
// 19 112 / 112, 399 x 9 x 399 154 / 196.  To 250 MB sides of 48: 201 x 33 x 201 124 / 137, 221 x
// 221 x 23 111 / 125, 221 x 29 x 221 130 / 157, 121 x 61 x 121 92 / 85.  To 600 MB of 72: 221 x
// 221 x 57 223 / 255, 221 x 73 x 221 283 / 293; but of 36 where the row fills 194 x 5
// tiles: 181 x 181 x 57 158 / 150, x 73 196 / 186.  Beyond, rows of 48 -- 17 x 301 x 301
// 277 / 384, 45 x 301 x 301 558 / 590, 53 x 301 x 301 606 / 597 -- and sides of 56 to 1 GB,
// of 19 above: 401 x 25 x 401 314 / 351, 301 x 301 x 49 355 / 366, 601 x 61 x 121 and 601 x
// 601 x 33 10 % less in one, 601 x 601 x 21 603 / 590.  FP64, rows of 36 and sides of
// 20: 33 x 301 x 301 606 / 618, 49 x 301 x 301 984 / 887; 301 x 301 x 19 270 / 282, x 23
// 314 / 303.
// So do planes so large that a run is cut below 8 (fine3_zcap; FP32, 33 planes:
// runs of 12 3908 / 3642, of 8 5225 / 5121; 17 planes: of 5 3933 / 4158, of 3 5043 /
// 5792, of 1 6099 / 9684).
template <typename S>
inline bool fine3_by_default(const Geo& g, double bytes) {
  const bool single = sizeof(S) == 4;
  if (bytes < (single ? 1e8 : 5e8) || fine3_zcap<S>(g) < 8) return false;
  const int n = g.nf[0] - 2, row = single ? (bytes < 6e8 ? 72 : 48) : 36;
  int side = single ? 19 : 20;
  if (single && bytes < 1e9) {
    if (bytes < 1.7e8 && n > 128 && !tall66(n, false)) side = 15;
    else if (bytes < 6e8) side = n >= 154 && n <= 192 ? 36 : (bytes < 2.5e8 ? 48 : 72);
    else side = 56;
  }
  return n >= row && std::min(g.nf[1], g.nf[2]) - 2 >= side;
}

// Default of the fine role of a D3Q19 H-RR level of `bytes` (two buffers):
// whether a substep runs in one marching pass (k_hrr3s) or as the velocity
// pass and the collision.  From 100 MB: us a step in two passes / in one,
// FP32 65^3 107 / 124, 97^3 211 / 182, 129^3 406 / 390.  Rows that use less than
// about 0.3 of a tile's columns (128, in double 64) keep the two passes: FP32
// 9 x 401 x 401 nodes 497 / 890, 17 x 301 x 301 406 / 588, 33 x 301 x 301 708 /
// 764, 37 x 301 x 301 757 / 776, 41 x 301 x 301 794 / 793, 45 x 301 x 301 850 / 819;
// FP64 9 x 401 x 401 984 / 1259, 17 x 301 x 301 816 / 873, 21 x 301 x 301 904 /
// 885, 21 x 181 x 181 286 / 306, 25 x 301 x 301 1004 / 944, 33 x 301 x 301 1159 /
// 1034.
template <typename S>
inline bool hrr3_fine_by_default(const Geo& g, double bytes) {
  return bytes >= 1e8 && g.nf[0] - 2 >= (sizeof(S) == 4 ? 40 : 18);
}

// The same for a D3Q19 H-RR coarse level (n[3] nodes): from 2 GB.  us a step in
// two passes / in one: FP32 256^3 844 / 736, 384 x 256 x 256 1210 / 1032, 1000 x 128 x
// 128 819 / 739; FP64 200^3 799 / 695, 96 x 280 x 280 762 / 669, 66 x 320 x 320 771 / 760.
// In FP32 rows that leave more than a fifth of the columns of two or three
// tiles of 128 idle keep the two passes: 194 x 280 x 280 822 / 857, 200 x 300 x 300 945 /
// 976, 260 x 256 x 256 893 / 930, 290 x 256 x 256 985 / 995.  Elsewhere one pass is level
// or ahead: 130 x 350 x 350 860 / 832, 160 x 320 x 320 829 / 715, 300 x 256 x 256 988 /
// 993, 300 x 1600 x 30 809 / 770, 390 x 240 x 240 1156 / 1121.
template <typename S>
inline bool hrr3_coarse_by_default(const int* n, double bytes) {
  if (bytes < 2e9) return false;
  return sizeof(S) == 8 || !((n[0] > 192 && n[0] < 205) || (n[0] > 256 && n[0] < 298));
}

// LDS variant (residency cap, kVarLds) of the H-RR collision in the two-pass
// form.  D3Q19: two work groups a CU, or three where variant 1 of an H-RR role
// asks for them; the other variants name tiles of the one-pass kernels and
// choose no cap where a level cannot take these (dynamic sigma, the coarse level
// of a nested grid's inner pair, planes past their addressing).  D2Q9, where only
// that coarse level has two passes: no cap (nested grid of 2048^2 / 2049^2 /
// 2049^2 nodes, us a step capped at two / not capped: FP32 595 / 576, FP64 1037 /
// 1027; 1024^2 FP64 355 / 352).
inline int hrr_cap(int D, int variant) { return D == 2 ? 0 : (variant == 1 ? 1 : 2); }

}  // namespace lbm
