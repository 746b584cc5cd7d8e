// d3q27.hpp -- device-side D3Q27 collision (OReg of Eq. (6) with D = 3, or
// lattice BGK of Eq. (1)) of one node in registers.
//
// The storage codecs, Coef64/Coeffs constants and helpers are those of the
// D2Q9 lattice (d2q9.hpp).  Algebraic forms used instead of the printed ones
// (identical in exact arithmetic):
//   * moments by lines: for each (c_y, c_z) the three populations along x
//     give their sum, difference and outer sum; planes of constant c_z
//     combine lines, the box combines planes (66 additions for rho, j and
//     the six second moments);
//   * both equilibria reproduce Pi^eq = rho theta I + rho u u, so the
//     trace-free stress of f^neq is the trace-free part of Pi - rho u u
//     (the shift w_i rho0 adds rho0 theta I, which has no trace-free part);
//   * with a trace-free S, (C C - C^2/3 I):S = sum_ab C_a C_b S_ab, and
//     kappa times it is assembled from per-axis tables:
//       A_a[c] = kappa S_aa C_a(c)^2,  T_ab[c] = 2 kappa S_ab C_a(c),
//       kappa b_i = (A_x + A_y + T_xy C_y) + A_z + (T_xz + T_yz) C_z;
//   * the guided equilibrium is rho X(c_x) Y(c_y) Z(c_z) with rest value +
//     small difference per axis factor, and in shifted storage
//     f^eq_i - w_i rho0 = drho XYZ + rho0 (dX YZ + a_x dY Z + a_x a_y dZ).
#pragma once

#include "d2q9.hpp"

namespace oreg {
namespace d3 {

// i = 9 (c_z + 1) + 3 (c_y + 1) + (c_x + 1).
__host__ __device__ constexpr int cx(int i) { return i % 3 - 1; }
__host__ __device__ constexpr int cy(int i) { return (i / 3) % 3 - 1; }
__host__ __device__ constexpr int cz(int i) { return i / 9 - 1; }
static_assert(cx(13) == 0 && cy(13) == 0 && cz(13) == 0, "rest velocity");
static_assert(cx(0) == -1 && cy(0) == -1 && cz(0) == -1 && cx(26) == 1 && cz(26) == 1, "corners");

// Rest weight of an axis component: a0 (c = 0) or a1 (c = +-1).
template <int c, typename R>
__host__ __device__ __forceinline__ R axis_w(const Coeffs<R>& k) {
  return c == 0 ? k.a0 : k.a1;
}

// Equilibrium of one node, population by population: feq_i (full value) and
// deq_i = feq_i - w_i rho0 (deq = feq when unshifted).  u2[a] = u_a^2.
//
// Guided: per-axis factors Psi(-1) = a1 + (u^2 - u)/2, Psi(0) = a0 - u^2,
// Psi(+1) = a1 + (u^2 + u)/2, as rest value + difference d[a][c + 1].
template <int EQ, typename R>
struct Factors {
  R d[3][3], F[3][3], rX[3];
  __host__ __device__ __forceinline__ Factors(R rho, const R (&u)[3], const R (&u2)[3],
                                              const Coeffs<R>& k) {
#pragma clang fp contract(off)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const R h = R(0.5) * u2[a];
      d[a][0] = fmadd(R(-0.5), u[a], h);
      d[a][1] = -u2[a];
      d[a][2] = fmadd(R(0.5), u[a], h);
      F[a][0] = k.a1 + d[a][0];
      F[a][1] = k.a0 + d[a][1];
      F[a][2] = k.a1 + d[a][2];
    }
#pragma unroll
    for (int ix = 0; ix < 3; ++ix) rX[ix] = rho * F[0][ix];
  }
  template <bool SHIFTED, int ix, int iy, int iz>
  __host__ __device__ __forceinline__ void at(R drho, R, const Coeffs<R>& k, R& feq, R& deq) const {
#pragma clang fp contract(off)
    feq = (rX[ix] * F[1][iy]) * F[2][iz];
    if constexpr (SHIFTED) {
      const R ax = ix == 1 ? k.a0 : k.a1, ay = iy == 1 ? k.a0 : k.a1;
      const R YZ = F[1][iy] * F[2][iz];
      const R XYZ = F[0][ix] * YZ;
      const R t3 = ((k.rho0 * ax) * ay) * d[2][iz];
      const R t2 = fmadd((k.rho0 * ax) * d[1][iy], F[2][iz], t3);
      deq = fmadd(drho, XYZ, fmadd(k.rho0 * d[0][ix], YZ, t2));
    } else {
      deq = feq;
    }
  }
};

// Polynomial equilibrium at theta0 = 1/3: rho W_i (1 + P_i),
// P_i = 3 c.u + 9/2 (c.u)^2 - 3/2 u^2.
template <typename R>
struct Factors<LB_EQ_POLY2, R> {
  R u[3], u2h;
  __host__ __device__ __forceinline__ Factors(R, const R (&v)[3], const R (&u2)[3],
                                              const Coeffs<R>&)
      : u{v[0], v[1], v[2]} {
#pragma clang fp contract(off)
    u2h = R(1.5) * ((u2[0] + u2[1]) + u2[2]);
  }
  template <bool SHIFTED, int ix, int iy, int iz>
  __host__ __device__ __forceinline__ void at(R drho, R rho, const Coeffs<R>& k, R& feq,
                                              R& deq) const {
#pragma clang fp contract(off)
    constexpr int ccx = ix - 1, ccy = iy - 1, ccz = iz - 1;
    R cu = R(0);
    if constexpr (ccx != 0) cu = ccx > 0 ? u[0] : -u[0];
    if constexpr (ccy != 0) cu = cu + (ccy > 0 ? u[1] : -u[1]);
    if constexpr (ccz != 0) cu = cu + (ccz > 0 ? u[2] : -u[2]);
    const R W = (axis_w<ccx>(k) * axis_w<ccy>(k)) * axis_w<ccz>(k);
    const R P = fmadd(cu, fmadd(R(4.5), cu, R(3)), -u2h);
    const R rW = rho * W;
    feq = fmadd(rW, P, rW);
    if constexpr (SHIFTED) deq = fmadd(drho, W, rW * P);
    else deq = feq;
  }
};

template <int EQ, bool SHIFTED, typename R>
__host__ __device__ __forceinline__ void equilibrium(R drho, R rho, const R (&u)[3],
                                                     const R (&u2)[3], const Coeffs<R>& k,
                                                     R (&feq)[27], R (&deq)[27]) {
  const Factors<EQ, R> fa(rho, u, u2, k);
  unroll<0, 27>([&](auto I) {
    constexpr int ix = cx(I.value) + 1, iy = cy(I.value) + 1, iz = cz(I.value) + 1;
    fa.template at<SHIFTED, ix, iy, iz>(drho, rho, k, feq[I.value], deq[I.value]);
  });
}

// What the OReg update keeps of a node's 27 populations: rho - rho0 (rho when
// unshifted), u, and the stress terms kappa S_aa (xx, yy, zz) and 2 kappa S_ab
// (xy, xz, yz) of the bracket of Eq. (6).  The post-collision populations are
// a function of these ten numbers alone (emit), so a node can be stored as
// them instead.
constexpr int kParams = 10;

// The six plane sums of the nine populations of one c_z, f[3 (c_y + 1) + (c_x +
// 1)]: density, x and y momentum, xx, yy and xy moments.
template <typename R>
struct PlaneSums {
  R P0, Px, Py, Pxx, Pyy, Pxy;
};
template <typename R>
__host__ __device__ __forceinline__ PlaneSums<R> plane_sums(const R (&f)[9]) {
#pragma clang fp contract(off)
  R L0[3], L1[3], L2[3];  // per line c_y
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    L2[l] = f[3 * l + 2] + f[3 * l];
    L0[l] = L2[l] + f[3 * l + 1];
    L1[l] = f[3 * l + 2] - f[3 * l];
  }
  PlaneSums<R> s;
  s.Pyy = L0[2] + L0[0];
  s.P0 = s.Pyy + L0[1];
  s.Py = L0[2] - L0[0];
  s.Px = (L1[2] + L1[0]) + L1[1];
  s.Pxy = L1[2] - L1[0];
  s.Pxx = (L2[2] + L2[0]) + L2[1];
  return s;
}

// rho - rho0 (rho when unshifted), j and the raw second moments M_ab = sum_i
// c_ia c_ib f_i (xx, yy, zz, xy, xz, yz) from the sums of the planes c_z = -1,
// 0, +1; `moments` does the same from all 27 populations of a node.
template <typename R>
__host__ __device__ __forceinline__ void combine(const PlaneSums<R>& m, const PlaneSums<R>& z,
                                                 const PlaneSums<R>& p, R& drho, R (&j)[3],
                                                 R (&M)[6]) {
#pragma clang fp contract(off)
  const R Mzz = p.P0 + m.P0;
  drho = Mzz + z.P0;
  j[0] = (p.Px + m.Px) + z.Px;
  j[1] = (p.Py + m.Py) + z.Py;
  j[2] = p.P0 - m.P0;
  M[0] = (p.Pxx + m.Pxx) + z.Pxx;
  M[1] = (p.Pyy + m.Pyy) + z.Pyy;
  M[2] = Mzz;
  M[3] = (p.Pxy + m.Pxy) + z.Pxy;
  M[4] = p.Px - m.Px;
  M[5] = p.Py - m.Py;
}

template <typename R>
__host__ __device__ __forceinline__ void moments(const R (&f)[27], R& drho, R (&j)[3],
                                                 R (&M)[6]) {
  PlaneSums<R> s[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    R g[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) g[i] = f[9 * c + i];
    s[c] = plane_sums(g);
  }
  combine(s[0], s[1], s[2], drho, j, M);
}

// The ten numbers of a node from its moments (OReg, any equilibrium).
template <bool SHIFTED, typename R>
__host__ __device__ __forceinline__ void reduce(R drho, const R (&j)[3], const R (&M)[6],
                                                const Coeffs<R>& k, R (&q)[kParams]) {
#pragma clang fp contract(off)
  const R rho = SHIFTED ? k.rho0 + drho : drho;
  const R inv = recip(rho);
  const R u[3] = {j[0] * inv, j[1] * inv, j[2] * inv};
  const R u2[3] = {u[0] * u[0], u[1] * u[1], u[2] * u[2]};
  // Trace-free part of Pi - rho u u (Pi^eq = rho theta I + rho u u).
  const R Dxx = fmadd(-rho, u2[0], M[0]);
  const R Dyy = fmadd(-rho, u2[1], M[1]);
  const R Dzz = fmadd(-rho, u2[2], M[2]);
  const R tr3 = ((Dxx + Dyy) + Dzz) * R(1.0 / 3.0);
  const R Sxx = Dxx - tr3, Syy = Dyy - tr3, Szz = Dzz - tr3;
  const R Sxy = fmadd(-rho, u[0] * u[1], M[3]);
  const R Sxz = fmadd(-rho, u[0] * u[2], M[4]);
  const R Syz = fmadd(-rho, u[1] * u[2], M[5]);
  const R kappa = k.kappa0 * inv;
  q[0] = drho;
  q[1] = u[0];
  q[2] = u[1];
  q[3] = u[2];
  q[4] = kappa * Sxx;
  q[5] = kappa * Syy;
  q[6] = kappa * Szz;
  q[7] = kappa * (Sxy + Sxy);
  q[8] = kappa * (Sxz + Sxz);
  q[9] = kappa * (Syz + Syz);
}

// The post-collision populations (shifted by w_i rho0 when SHIFTED) from the
// ten numbers, handed to put(i, f_i) nine at a time (one c_y), with an
// ordering point (next()) before each c_y: only one c_y's factors are alive at
// a time, where evaluating all 27 equilibria first takes 54 more registers in
// FP64.
template <int EQ, bool SHIFTED, typename R, class Put, class Next>
__host__ __device__ __forceinline__ void emit_each(const R (&q)[kParams], const Coeffs<R>& k,
                                                   Put&& put, Next&& next) {
#pragma clang fp contract(off)
  const R drho = q[0], rho = SHIFTED ? k.rho0 + drho : drho;
  const R u[3] = {q[1], q[2], q[3]};
  const R u2[3] = {u[0] * u[0], u[1] * u[1], u[2] * u[2]};
  const R kxx = q[4], kyy = q[5], kzz = q[6], txy = q[7], txz = q[8], tyz = q[9];
  const Factors<EQ, R> fa(rho, u, u2, k);
  R Ax[3], Txy[3], Txz[3], Cz[3], Az[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const R Cx = R(c - 1) - u[0];
    Ax[c] = (kxx * Cx) * Cx;
    Txy[c] = txy * Cx;
    Txz[c] = txz * Cx;
    Cz[c] = R(c - 1) - u[2];
    Az[c] = (kzz * Cz[c]) * Cz[c];
  }
  unroll<0, 3>([&](auto IY) {
    constexpr int iy = IY.value;
    next();
    const R Cy = R(iy - 1) - u[1];
    const R Ay = (kyy * Cy) * Cy, Tyz = tyz * Cy;
    unroll<0, 3>([&](auto IX) {
      constexpr int ix = IX.value;
      const R B = fmadd(Txy[ix], Cy, Ax[ix] + Ay);
      const R U = Txz[ix] + Tyz;
      unroll<0, 3>([&](auto IZ) {
        constexpr int iz = IZ.value, i = 9 * iz + 3 * iy + ix;
        R feq, deq;
        fa.template at<SHIFTED, ix, iy, iz>(drho, rho, k, feq, deq);
        const R term = fmadd(U, Cz[iz], B + Az[iz]);
        put(std::integral_constant<int, i>{}, fmadd(feq, term, deq));
      });
    });
  });
}

template <int EQ, bool SHIFTED, typename R>
__host__ __device__ __forceinline__ void emit(const R (&q)[kParams], const Coeffs<R>& k,
                                              R (&f)[27]) {
  emit_each<EQ, SHIFTED>(q, k, [&](auto I, R v) { f[I.value] = v; }, [] {});
}

// Collide one node in place: f holds the pre-collision populations (shifted
// by w_i rho0 when SHIFTED) and receives the post-collision ones.
template <int EQ, int COLL, bool SHIFTED, typename R>
__host__ __device__ __forceinline__ void collide(R (&f)[27], const Coeffs<R>& k) {
#pragma clang fp contract(off)
  R drho, j[3], M[6];
  moments(f, drho, j, M);
  if constexpr (COLL == LB_COLL_BGK) {
    const R rho = SHIFTED ? k.rho0 + drho : drho;
    const R inv = recip(rho);
    const R u[3] = {j[0] * inv, j[1] * inv, j[2] * inv};
    const R u2[3] = {u[0] * u[0], u[1] * u[1], u[2] * u[2]};
    R feq[27], deq[27];
    equilibrium<EQ, SHIFTED>(drho, rho, u, u2, k, feq, deq);
    unroll<0, 27>([&](auto I) { f[I.value] = fmadd(k.omega, deq[I.value] - f[I.value], f[I.value]); });
  } else {
    R q[kParams];
    reduce<SHIFTED>(drho, j, M, k, q);
    emit<EQ, SHIFTED>(q, k, f);
  }
}

// Rest weight times rho0 of a population with velocity (cx, cy, cz), FP64.
__host__ __device__ __forceinline__ double shift64(int vx, int vy, int vz, const Coef64& c) {
  auto w = [&](int v) { return v == 0 ? c.a0 : c.a1; };
  return w(vx) * w(vy) * w(vz) * c.rho0;
}

}  // namespace d3
}  // namespace oreg
