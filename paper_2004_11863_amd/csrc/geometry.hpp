// geometry.hpp -- two-level grid geometry and node classes (host and device).
//
// The fine patch is the box [a, a+m] of coarse vertices; fine node j sits at
// coarse coordinate a + j/2, so the fine level has 2m+1 nodes per axis and
// its outer layer (j = 0 or 2m) is the overlap ring of Fig. Overlap.  The
// classes follow that figure, written for a closed patch:
//   coarse TF  : coarse vertices on the boundary of [a, a+m]      (c -> f)
//   coarse TN  : coarse vertices on the boundary of [a+1, a+m-1]  (f -> c)
//   covered    : coarse vertices inside [a+1, a+m-1] (not evolved)
//   fine TF    : ring nodes co-located with a coarse vertex
//   fine IE    : other ring nodes (one half-integer coordinate)
//   fine IEFACE: 3D ring nodes with two half-integer coordinates
//   fine TN    : fine nodes co-located with coarse TN nodes
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace lbm {

enum CoarseClass : int { CC_MIDDLE = 0, CC_TF = 1, CC_TN = 2, CC_COVERED = 3 };
enum FineClass : int { FC_MIDDLE = 0, FC_TF = 1, FC_IE = 2, FC_IEFACE = 3, FC_TN = 4 };

// Device arrays use a padded row pitch (pc, pf: nodes per row rounded up to
// a multiple of 4, or in large three-dimensional fine levels to whole
// 128-byte lines, fine_pitch in lbm.hip) so every row starts aligned; Ncp, Nfp are the
// padded node counts of a level (the positions of pop_at below, and the plane
// size of the velocity planes).  Nc, Nf count logical nodes (the x-fastest
// order of the C ABI and of the interface tables).  (A power-of-two fine
// pitch, which keeps rows inside one storage block, was measured slower: rows
// a power of two apart share HBM channels.)
struct Geo {
  int D;
  int n[3];   // coarse nodes per axis (1 on unused axes)
  int a[3];   // patch lower corner (coarse vertex)
  int m[3];   // patch size in coarse cells
  int nf[3];  // fine nodes per axis (2m+1; 1 on unused axes or without patch)
  int has_fine;
  int64_t Nc, Nf;
  int pc, pf;        // row pitch of coarse / fine device arrays
  int fxo;           // offset of fine node x = 0 inside its row: the first
                     // middle node (x = 1) starts a 16-byte (or line) boundary
  int64_t Ncp, Nfp;  // padded plane sizes
};

constexpr int kPitchAlign = 4;
__host__ __device__ inline int pitch_of(int nx) { return (nx + kPitchAlign - 1) / kPitchAlign * kPitchAlign; }

// Padded device offset of a coarse / fine node.
__host__ __device__ inline int64_t cpos(const Geo& g, int x, int y, int z) {
  return (int64_t)x + (int64_t)g.pc * ((int64_t)y + (int64_t)g.n[1] * z);
}
__host__ __device__ inline int64_t fpos(const Geo& g, int x, int y, int z) {
  return (int64_t)(x + g.fxo) + (int64_t)g.pf * ((int64_t)y + (int64_t)g.nf[1] * z);
}
// Logical node index -> coordinates (32-bit: levels of 2^31 or more positions
// are rejected, and 64-bit divisions cost the interface kernels some hundred
// instructions a node).
__host__ __device__ inline void decode_in(const int* n, int64_t i, int& x, int& y, int& z) {
  const uint32_t k = (uint32_t)i, r = k / (uint32_t)n[0];
  x = (int)(k - r * (uint32_t)n[0]);
  z = (int)(r / (uint32_t)n[1]);
  y = (int)(r - (uint32_t)z * (uint32_t)n[1]);
}
__host__ __device__ inline void cdecode(const Geo& g, int64_t i, int& x, int& y, int& z) { decode_in(g.n, i, x, y, z); }
__host__ __device__ inline void fdecode(const Geo& g, int64_t i, int& x, int& y, int& z) { decode_in(g.nf, i, x, y, z); }

__host__ __device__ inline int coarse_class(const Geo& g, int x, int y, int z) {
  if (!g.has_fine) return CC_MIDDLE;
  const int c[3] = {x, y, z};
  bool in_tn = true, on_tn = false, in_tf = true, on_tf = false;
  for (int d = 0; d < g.D; ++d) {
    const int lo = g.a[d], hi = g.a[d] + g.m[d];
    if (c[d] < lo + 1 || c[d] > hi - 1) in_tn = false;
    if (c[d] == lo + 1 || c[d] == hi - 1) on_tn = true;
    if (c[d] < lo || c[d] > hi) in_tf = false;
    if (c[d] == lo || c[d] == hi) on_tf = true;
  }
  if (in_tn) return on_tn ? CC_TN : CC_COVERED;
  return (in_tf && on_tf) ? CC_TF : CC_MIDDLE;
}

__host__ __device__ inline bool fine_is_ring(const Geo& g, int x, int y, int z) {
  return x == 0 || x == g.nf[0] - 1 || y == 0 || y == g.nf[1] - 1 ||
         (g.D == 3 && (z == 0 || z == g.nf[2] - 1));
}

__host__ __device__ inline int fine_class(const Geo& g, int x, int y, int z) {
  const int j[3] = {x, y, z};
  int odd = 0;
  bool even = true, in_tn = true, on_tn = false;
  for (int d = 0; d < g.D; ++d) {
    const int M = g.nf[d] - 1;
    if (j[d] & 1) {
      odd++;
      even = false;
    }
    if (j[d] < 2 || j[d] > M - 2) in_tn = false;
    if (j[d] == 2 || j[d] == M - 2) on_tn = true;
  }
  if (fine_is_ring(g, x, y, z)) return odd == 0 ? FC_TF : (odd == 1 ? FC_IE : FC_IEFACE);
  return (even && in_tn && on_tn) ? FC_TN : FC_MIDDLE;
}

// History entry of the coarse vertex (X, Y, Z) - 1 of a three-dimensional patch
// (offsets from its lower corner, so X, Y, Z in [0, m + 2]) that lies on a face
// plane: the closed form of the table's order (coarse node order over the face
// planes within one vertex of the patch).  A z plane holds all (m0 + 3)(m1 + 3)
// vertices where it is a face plane, else rows of m0 + 3 on the y face planes
// and of two vertices elsewhere.
__host__ __device__ inline int hist3_index(const Geo& g, int X, int Y, int Z) {
  const int row = g.m[0] + 3, full = row * (g.m[1] + 3), rim = 2 * row + 2 * (g.m[1] + 1);
  const int base = Z * rim + (full - rim) * ((Z > 1 ? 1 : 0) + (Z > g.m[2] + 1 ? 1 : 0));
  if (Z == 1 || Z == g.m[2] + 1) return base + Y * row + X;
  const int r = base + 2 * Y + (row - 2) * ((Y > 1 ? 1 : 0) + (Y > g.m[1] + 1 ? 1 : 0));
  return Y == 1 || Y == g.m[1] + 1 ? r + X : r + (X == 1 ? 0 : 1);
}
// Tiles of kRingU x kRingV ring nodes on the six faces of a three-dimensional
// patch (normal axis w; a z face holds its edges, a y face its x edges).  (pick
// evaluates both values: loads behind a branch on w are merged into one load
// from a chosen address, which puts the geometry in scratch memory.)
__host__ __device__ inline int pick(bool c, int a, int b) { return c ? a : b; }
constexpr int kRingU = 32, kRingV = 8;
__host__ __device__ inline int ring3_nu(const Geo& g, int w) { return pick(w == 0, g.nf[1], g.nf[0]); }
__host__ __device__ inline int ring3_nv(const Geo& g, int w) { return pick(w == 2, g.nf[1], g.nf[2]); }
__host__ __device__ inline int ring3_face_tiles(const Geo& g, int w) {
  return ((ring3_nu(g, w) + kRingU - 1) / kRingU) * ((ring3_nv(g, w) + kRingV - 1) / kRingV);
}
__host__ __device__ inline int ring3_tiles(const Geo& g) {
  return 2 * (ring3_face_tiles(g, 0) + ring3_face_tiles(g, 1) + ring3_face_tiles(g, 2));
}
// Vertex patch of a tile: the stencils reach from one vertex before its first
// node's to two past its last.
constexpr int kRingPU = kRingU / 2 + 3, kRingPV = kRingV / 2 + 3;
// Face, side and first node of tile t; false past the last tile.
__host__ __device__ inline bool ring3_tile(const Geo& g, int t, int& w, int& side, int& u0, int& v0) {
  const int n2 = ring3_face_tiles(g, 2), n1 = ring3_face_tiles(g, 1), n0 = ring3_face_tiles(g, 0);
  int n;
  if (t < 2 * n2) {
    w = 2;
    n = n2;
  } else if (t < 2 * (n2 + n1)) {
    w = 1;
    n = n1;
    t -= 2 * n2;
  } else if (t < 2 * (n2 + n1 + n0)) {
    w = 0;
    n = n0;
    t -= 2 * (n2 + n1);
  } else {
    return false;
  }
  side = t / n;
  t -= side * n;
  const int tu = (ring3_nu(g, w) + kRingU - 1) / kRingU, iv = t / tu;
  u0 = (t - iv * tu) * kRingU;
  v0 = iv * kRingV;
  return true;
}
// History entry of vertex (pu, pv) of the patch of a tile, or -1 outside the
// history set.
__host__ __device__ inline int ring3_vertex(const Geo& g, int w, int side, int u0, int v0, int pu, int pv) {
  const int mu = pick(w == 0, g.m[1], g.m[0]), mv = pick(w == 2, g.m[1], g.m[2]);
  const int U = u0 / 2 + pu, V = v0 / 2 + pv;  // (vertex + 1)
  if (U > mu + 2 || V > mv + 2) return -1;
  const int mw = pick(w == 2, g.m[2], pick(w == 1, g.m[1], g.m[0])), W = side == 0 ? 1 : mw + 1;
  return hist3_index(g, pick(w == 0, W, U), pick(w == 0, U, pick(w == 1, W, V)), pick(w == 2, W, V));
}

// Compact copy of the fine state in the two x-normal bands of the patch,
// x in [0, 4] (side 0) and [nx - 5, nx - 1] (side 1), five nodes per row:
// [side][population][z][y][x offset].  In the row-major layout every
// population of those nodes fills its own cache line; here consecutive rows
// are 5 values apart.  (The bands overlap when nx < 10: a node may sit on
// both sides.)
__host__ __device__ inline int64_t xband_at(const Geo& g, int Q, int side, int q, int y, int z, int xo) {
  return ((((int64_t)side * Q + q) * g.nf[2] + z) * g.nf[1] + y) * 5 + xo;
}
__host__ __device__ inline int64_t xband_elems(const Geo& g, int Q) { return (int64_t)2 * Q * g.nf[2] * g.nf[1] * 5; }

// Periodic wrap of a coarse coordinate displaced by at most one period.
__host__ __device__ inline int wrap(int x, int n) { return x < 0 ? x + n : (x >= n ? x - n : x); }

// Population storage, array of structure-of-arrays: the padded node positions
// p of a level are cut into blocks of PB consecutive positions; block b holds
// Q sub-blocks of 32 KB, one per population, each with the PB values of that
// block.  A pull-stream step then keeps its 2Q concurrent memory streams
// within two windows of Q x 32 KB instead of 2Q planes spread over the whole
// buffer, which HBM serves markedly faster than plain structure-of-arrays.
template <typename S>
struct PopBlock {
  static constexpr int SHIFT = sizeof(S) == 4 ? 13 : 12;  // 8192 floats or 4096 doubles
  static constexpr int64_t B = (int64_t)1 << SHIFT;
};
// Written as base(p) + q B, base(p) = p + (Q - 1) B floor(p / B), which is
// ((p / B) Q + q) B + p mod B: the Q populations of a node share base(p).
template <typename S, int Q>
__host__ __device__ inline int64_t pop_at(int64_t p, int q) {
  constexpr int SH = PopBlock<S>::SHIFT;
  constexpr int64_t B = PopBlock<S>::B;
  return p + (int64_t)(Q - 1) * B * (p >> SH) + (int64_t)q * B;
}
// Elements of a population buffer for NP padded positions: whole blocks up
// to and including position NP (the last x-vector of a fine row reaches one
// position past the end of its row).
template <typename S>
__host__ __device__ inline int64_t pop_elems(int64_t NP, int Q) {
  return ((NP >> PopBlock<S>::SHIFT) + 1) * (int64_t)Q * PopBlock<S>::B;
}

}  // namespace lbm
