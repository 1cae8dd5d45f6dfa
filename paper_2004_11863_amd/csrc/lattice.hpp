// lattice.hpp -- lattice tables and per-node physics of the two-level LBM
// hot path (device side, gfx950).
//
// Everything here is written for unrolled loops over the populations: the
// velocity components are constexpr functions of the population index, so
// after unrolling every Hermite polynomial value folds into an immediate.
//
// Populations are handled in "stored form": s_i = f_i - DEV * w_i.  With
// DEV = 0 the stored value is the population itself (FP64 path); with DEV = 1
// it is the deviation from the rest state (FP32 deviation path), which keeps
// the single-precision significand for the O(Ma) part of f.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace lbm {

// Compile-time loop: f(std::integral_constant<int, I>) for I = 0 .. N-1.
template <int N, int I = 0, typename F>
__host__ __device__ inline void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// ---------------------------------------------------------------------------
// Lattices.  D2Q9 in the order of Sec. 3.1 (eq xi_i, eq w_i).  D3Q19 is the
// standard 19-velocity lattice: rest, +-x, +-y, +-z, then (+-1,+-1,0),
// (+-1,0,+-1), (0,+-1,+-1) in the order (1,1), (-1,-1), (1,-1), (-1,1).
template <int LAT>
struct Lattice;

template <>
struct Lattice<0> {
  static constexpr int D = 2, Q = 9;
  __host__ __device__ static constexpr int cx(int i) {
    return (i == 1 || i == 5 || i == 8) ? 1 : ((i == 3 || i == 6 || i == 7) ? -1 : 0);
  }
  __host__ __device__ static constexpr int cy(int i) {
    return (i == 2 || i == 5 || i == 6) ? 1 : ((i == 4 || i == 7 || i == 8) ? -1 : 0);
  }
  __host__ __device__ static constexpr int cz(int) { return 0; }
  __host__ __device__ static constexpr double w(int i) {
    return i == 0 ? 4.0 / 9.0 : (i < 5 ? 1.0 / 9.0 : 1.0 / 36.0);
  }
};

template <>
struct Lattice<1> {
  static constexpr int D = 3, Q = 19;
  __host__ __device__ static constexpr int cx(int i) {
    return (i == 1 || i == 7 || i == 9 || i == 11 || i == 13) ? 1
           : ((i == 2 || i == 8 || i == 10 || i == 12 || i == 14) ? -1 : 0);
  }
  __host__ __device__ static constexpr int cy(int i) {
    return (i == 3 || i == 7 || i == 10 || i == 15 || i == 17) ? 1
           : ((i == 4 || i == 8 || i == 9 || i == 16 || i == 18) ? -1 : 0);
  }
  __host__ __device__ static constexpr int cz(int i) {
    return (i == 5 || i == 11 || i == 14 || i == 15 || i == 18) ? 1
           : ((i == 6 || i == 12 || i == 13 || i == 16 || i == 17) ? -1 : 0);
  }
  __host__ __device__ static constexpr double w(int i) {
    return i == 0 ? 1.0 / 3.0 : (i < 7 ? 1.0 / 18.0 : 1.0 / 36.0);
  }
};

// Number of independent strain-rate components kept: xx, yy, xy (2D) or
// xx, yy, zz, xy, xz, yz (3D).
template <int D>
struct NS {
  static constexpr int value = D == 2 ? 3 : 6;
};

// Symmetric second-order tensor, components xx, yy, zz, xy, xz, yz.
template <typename T>
struct Sym {
  T xx, yy, zz, xy, xz, yz;
};

// ---------------------------------------------------------------------------
// Per-node physics in moment space.
//
// Every population the scheme produces (equilibrium, BGK or regularised
// post-collision state) is a polynomial in the lattice velocity,
//   s_i = w_i [ A + xi_i.J + xi_i xi_i : M + sum_P H_P(xi_i) K_P ],
// where the H_P are the third-order Hermite polynomials the lattice carries
// (D2Q9: H_xxy, H_xyy; D3Q19: the sums and differences of the pairs
// (H_xxy, H_yzz), (H_xzz, H_xyy), (H_yyz, H_xxz)).  The node computes a few
// coefficients once and evaluates opposite velocities together: the even part
// A + xi xi : M is shared, the odd part flips sign (build()).
//
// The bulk kernels issue as much arithmetic as they move bytes (k_fine2 keeps
// the vector ALU 65-76 % busy), so the collision is written for few
// operations: the momentum j is used as summed (never rho times u again), the
// products t_ab = j_a u_b serve the equilibrium, the non-equilibrium moment
// and the third order, the weights are folded into the coefficients, and the
// third-order terms are taken per plane (on a diagonal of plane (a, b) only
// K_aab and K_abb remain of the sums and differences).
template <int LAT, bool DEV, typename T>
struct Node {
  using L = Lattice<LAT>;
  static constexpr int Q = L::Q;
  static constexpr int D = L::D;

  // index of the opposite velocity
  __host__ __device__ static constexpr int opp(int i) {
    for (int j = 0; j < Q; ++j)
      if (L::cx(j) == -L::cx(i) && L::cy(j) == -L::cy(i) && L::cz(j) == -L::cz(i)) return j;
    return i;
  }
  // eqs moment_rho, moment_rhoU.  r0: sum of stored values (rho for DEV = 0,
  // rho - 1 for DEV = 1).  Opposite velocities enter as the pair sum (even
  // moments) and the pair difference (odd moments); sums start from -0, which
  // the compiler folds away (x + -0 = x exactly).
  __device__ __host__ static __forceinline__ void moments(const T* s, T& rho, T& r0, T* j, T* u) {
    T m = s[0], jx = T(-0.0), jy = T(-0.0), jz = T(-0.0);
    static_for<Q>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      constexpr int j = opp(i);
      if constexpr (i != 0 && i < j) {
        const T p = s[i] + s[j], d = s[i] - s[j];
        m += p;
        if constexpr (L::cx(i) > 0) jx += d;
        if constexpr (L::cx(i) < 0) jx -= d;
        if constexpr (L::cy(i) > 0) jy += d;
        if constexpr (L::cy(i) < 0) jy -= d;
        if constexpr (D == 3 && L::cz(i) > 0) jz += d;
        if constexpr (D == 3 && L::cz(i) < 0) jz -= d;
      }
    });
    r0 = m;
    rho = DEV ? T(1) + m : m;
    const T ir = T(1) / rho;
    j[0] = jx;
    j[1] = jy;
    j[2] = (D == 3) ? jz : T(0);
    u[0] = jx * ir;
    u[1] = jy * ir;
    u[2] = (D == 3) ? jz * ir : T(0);
  }
  __device__ __host__ static __forceinline__ void moments(const T* s, T& rho, T& r0, T* u) {
    T j[3];
    moments(s, rho, r0, j, u);
  }

  // Second moments Pi_ab = sum_i xi_a xi_b s_i, from the pair sums (xi_a xi_b
  // is the same for opposite velocities).
  __device__ __host__ static __forceinline__ Sym<T> second(const T* s) {
    T pxx = T(-0.0), pyy = T(-0.0), pzz = T(-0.0), pxy = T(-0.0), pxz = T(-0.0), pyz = T(-0.0);
    static_for<Q>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      constexpr int j = opp(i);
      if constexpr (i != 0 && i < j) {
        constexpr int x = L::cx(i), y = L::cy(i), z = L::cz(i);
        const T p = s[i] + s[j];
        if constexpr (x != 0) pxx += p;
        if constexpr (y != 0) pyy += p;
        if constexpr (D == 3 && z != 0) pzz += p;
        if constexpr (x * y > 0) pxy += p;
        if constexpr (x * y < 0) pxy -= p;
        if constexpr (D == 3 && x * z > 0) pxz += p;
        if constexpr (D == 3 && x * z < 0) pxz -= p;
        if constexpr (D == 3 && y * z > 0) pyz += p;
        if constexpr (D == 3 && y * z < 0) pyz -= p;
      }
    });
    if constexpr (D == 2) pzz = pxz = pyz = T(0);
    return Sym<T>{pxx, pyy, pzz, pxy, pxz, pyz};
  }

  // j_a u_b = rho u_a u_b.
  __device__ __host__ static __forceinline__ Sym<T> flux(const T* j, const T* u) {
    Sym<T> t;
    t.xx = j[0] * u[0];
    t.yy = j[1] * u[1];
    t.xy = j[0] * u[1];
    t.zz = D == 3 ? j[2] * u[2] : T(0);
    t.xz = D == 3 ? j[0] * u[2] : T(0);
    t.yz = D == 3 ? j[1] * u[2] : T(0);
    return t;
  }

  // All Q stored values of f0 + om f1^RR (eqs fEqO3, f1RR, a13RR) from r0, the
  // momentum j, the velocity u, t = flux(j, u) and m = t + om a1^(2):
  //   A = r0 - 3/2 tr m,  J = 3 j,  M = 9/2 m,
  //   third order rho u_a u_a u_b + om a1^(3)_aab = 2 u_a m_ab + u_b (m_aa - 2 t_aa)
  // (eq a13RR: a1^(3)_aab = 2 u_a a1_ab + u_b a1_aa).  EQ: the equilibrium
  // alone, m = t, where the third order is u_b t_aa.
  // With w = 1/36 on every two-axis velocity the value there is
  //   A/36 + (M_aa + M_bb)/36 +- m_ab/4 +- (g_a +- g_b),  g_a = j_a/12 + K_abb/4,
  // M_aa/36 = m_aa/8; the even part of the one-axis velocities is 4 (D2Q9) or
  // 2 (D3Q19) times (A + M_aa)/36.  The rest population and the odd part of
  // the one-axis velocities are taken as what is left of r0 and j: the
  // factors 1/36 and 1/12 are not exact in binary, and with a rounded factor
  // on every velocity the same relative error would enter the mass and the
  // momentum at every collision.
  template <bool EQ>
  __device__ __host__ static __forceinline__ void build(T r0, const T* j, const T* u, const Sym<T>& t,
                                                        const Sym<T>& m, T* out) {
    const T B = r0 - T(1.5) * (D == 3 ? m.xx + m.yy + m.zz : m.xx + m.yy);
    const T A = B * T(1.0 / 36.0);
    const T nx = T(0.125) * m.xx, ny = T(0.125) * m.yy, nz = T(0.125) * m.zz;
    const T jx = T(1.0 / 12.0) * j[0], jy = T(1.0 / 12.0) * j[1], jz = T(1.0 / 12.0) * j[2];
    // K_aab = 2 u_a m_ab + u_b q_aa
    const T qx = EQ ? t.xx : m.xx - T(2) * t.xx, qy = EQ ? t.yy : m.yy - T(2) * t.yy;
    const T qz = EQ ? t.zz : m.zz - T(2) * t.zz;
    const T vx = T(2) * u[0], vy = T(2) * u[1], vz = T(2) * u[2];
    auto third = [](T va, T mab, T ub, T qa) __attribute__((always_inline)) { return EQ ? ub * qa : va * mab + ub * qa; };
    // g_a of plane (a, b) from K_abb
    auto odd = [](T ja, T kabb) __attribute__((always_inline)) { return ja + T(0.25) * kabb; };
    // one-axis velocities along a (i, its opposite o): r times the even part
    // e, the odd part o
    auto axis = [&](T r, T e, T o, int i, int io) __attribute__((always_inline)) {
      out[i] = r * e + o;
      out[io] = r * e - o;
    };
    // two-axis velocities of plane (a, b): p (+,+), its opposite, q (+,-),
    // its opposite
    auto plane = [&](T na, T nb, T mab, T ga, T gb, int p, int po, int q, int qo) __attribute__((always_inline)) {
      const T e = A + na + nb;
      const T ep = e + T(0.25) * mab, eq = e - T(0.25) * mab;
      const T op = ga + gb, oq = ga - gb;
      out[p] = ep + op;
      out[po] = ep - op;
      out[q] = eq + oq;
      out[qo] = eq - oq;
    };
    if constexpr (D == 2) {
      const T gx = odd(jx, third(vy, m.xy, u[0], qy)), gy = odd(jy, third(vx, m.xy, u[1], qx));
      out[0] = B - T(20) * A;
      axis(T(4), A + nx, T(0.5) * j[0] - T(2) * gx, 1, 3);
      axis(T(4), A + ny, T(0.5) * j[1] - T(2) * gy, 2, 4);
      plane(nx, ny, m.xy, gx, gy, 5, 7, 8, 6);
    } else {
      const T gxy = odd(jx, third(vy, m.xy, u[0], qy)), gxz = odd(jx, third(vz, m.xz, u[0], qz));
      const T gyx = odd(jy, third(vx, m.xy, u[1], qx)), gyz = odd(jy, third(vz, m.yz, u[1], qz));
      const T gzx = odd(jz, third(vx, m.xz, u[2], qx)), gzy = odd(jz, third(vy, m.yz, u[2], qy));
      out[0] = B - T(24) * A;
      axis(T(2), A + nx, T(0.5) * j[0] - T(2) * (gxy + gxz), 1, 2);
      axis(T(2), A + ny, T(0.5) * j[1] - T(2) * (gyx + gyz), 3, 4);
      axis(T(2), A + nz, T(0.5) * j[2] - T(2) * (gzx + gzy), 5, 6);
      plane(nx, ny, m.xy, gxy, gyx, 7, 8, 9, 10);
      plane(nx, nz, m.xz, gxz, gzx, 11, 12, 13, 14);
      plane(ny, nz, m.yz, gyz, gzy, 15, 16, 17, 18);
    }
  }

  // t + om a, componentwise.
  __device__ __host__ static __forceinline__ Sym<T> relaxed(const Sym<T>& t, T om, const Sym<T>& a) {
    Sym<T> m;
    m.xx = t.xx + om * a.xx;
    m.yy = t.yy + om * a.yy;
    m.xy = t.xy + om * a.xy;
    m.zz = D == 3 ? t.zz + om * a.zz : T(0);
    m.xz = D == 3 ? t.xz + om * a.xz : T(0);
    m.yz = D == 3 ? t.yz + om * a.yz : T(0);
    return m;
  }

  // Stored values of f0(rho, u) + om f1^RR(a) from given rho, u and a1^(2) = a.
  __device__ __host__ static __forceinline__ void regular(T rho, T r0, const T* u, T om, const Sym<T>& a, T* out) {
    const T j[3] = {rho * u[0], rho * u[1], D == 3 ? rho * u[2] : T(0)};
    const Sym<T> t = flux(j, u);
    build<false>(r0, j, u, t, relaxed(t, om, a), out);
  }

  // Stored-form equilibrium s0_i = f0_i - DEV w_i (eq fEqO3 and its D3Q19
  // counterpart).
  __device__ __host__ static __forceinline__ void feq(T rho, T r0, const T* u, T* out) {
    const T j[3] = {rho * u[0], rho * u[1], D == 3 ? rho * u[2] : T(0)};
    const Sym<T> t = flux(j, u);
    build<true>(r0, j, u, t, t, out);
  }

  // Collision of one node, in place on stored populations s[Q].
  //   model 0 (BGK, eq BGKmodel):      s* = s0 + om (s - s0)
  //   model 1 (RR,  eq LBMscheme_reg): s* = s0 + om f1RR(a1)
  //   model 2 (H-RR, eq a1ij_HRR):     a1 <- sig a1 + (1 - sig)(-2 tau rho c_s^2 S)
  // om = 1 - 1/tau.  With the third-order equilibrium,
  // sum_i xi xi f0_i = rho (u u + c_s^2 I), so a1 = Pi - r0/3 I - rho u u
  // in stored form (the rest state carries Pi = I/3).
  __device__ __host__ static __forceinline__ void collide(T* s, int model, T om, T tau, T sig, const Sym<T>* S) {
    T rho, r0, j[3], u[3];
    moments(s, rho, r0, j, u);
    const Sym<T> t = flux(j, u);
    if (model == 0) {
      T s0[Q];
      build<true>(r0, j, u, t, t, s0);
#pragma unroll
      for (int i = 0; i < Q; ++i) s[i] = s0[i] + om * (s[i] - s0[i]);
      return;
    }
    const Sym<T> P = second(s);
    const T tr0 = r0 * T(1.0 / 3.0);
    Sym<T> a;
    a.xx = (P.xx - tr0) - t.xx;
    a.yy = (P.yy - tr0) - t.yy;
    a.zz = (D == 3) ? (P.zz - tr0) - t.zz : T(0);
    a.xy = P.xy - t.xy;
    a.xz = (D == 3) ? P.xz - t.xz : T(0);
    a.yz = (D == 3) ? P.yz - t.yz : T(0);
    if (model == 2) {
      const T k = (T(1) - sig) * (T(-2.0 / 3.0) * tau * rho);
      a.xx = sig * a.xx + k * S->xx;
      a.yy = sig * a.yy + k * S->yy;
      a.xy = sig * a.xy + k * S->xy;
      if (D == 3) {
        a.zz = sig * a.zz + k * S->zz;
        a.xz = sig * a.xz + k * S->xz;
        a.yz = sig * a.yz + k * S->yz;
      }
    }
    build<false>(r0, j, u, t, relaxed(t, om, a), s);
  }
};

}  // namespace lbm
