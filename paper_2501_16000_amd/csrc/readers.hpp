// readers.hpp -- what a node's readers (moments, diagnostics, profile, export) take
// from a buffer: its pre-collision populations and their sums.
#pragma once

#include "dispatch.hpp"

namespace oreg {
namespace {
using namespace detail;

// Readers take a lattice's equilibrium (NEQ) where its buffers may
// hold the five numbers of a node (d2q9.hpp: Params) instead of populations,
// as the format flag *fmt says; kPopsOnly otherwise (fmt unused).
constexpr int kPopsOnly = -1;
template <int NEQ>
__device__ __forceinline__ bool holds_numbers(const unsigned int* __restrict__ fmt) {
  if constexpr (NEQ == kPopsOnly) return false;
  else return *fmt != 0;
}

// Population I that node (xs, ys) sends out, from its five numbers: emit with
// the eight others dropped by the compiler.
template <int NEQ, int ST, int I>
__device__ __forceinline__ typename Storage<ST>::T emitted(const typename Storage<ST>::T* __restrict__ src,
                                                           const Geometry& g, int xs, int ys,
                                                           const Coeffs<typename Storage<ST>::R>& k) {
  using S = Storage<ST>;
  const typename S::T* const q = src + (int64_t)ys * g.nx + xs;
  typename S::R f[9];
  emit<NEQ, S::shifted>(Params<typename S::R>{q[0], q[g.plane], q[2 * g.plane], q[3 * g.plane],
                                              q[4 * g.plane]},
                        k, f);
  return S::store(f[I]);
}

// Pre-collision populations of node (x, y) in FP64, still shifted by w_i rho0.
template <int ST, int NEQ>
__device__ __forceinline__ void gather64(const typename Storage<ST>::T* __restrict__ src,
                                         const Geometry& g, int x, int y, const Coef64& c,
                                         bool numbers, double (&d)[9]) {
  using S = Storage<ST>;
  const int xm = wrap_dec(x, g.nx), xp = wrap_inc(x, g.nx);
  const int ym = wrap_dec(y, g.ny), yp = wrap_inc(y, g.ny);
  if constexpr (NEQ != kPopsOnly) {
    if (numbers) {
      const Coeffs<typename S::R> k(c);
      unroll<0, 9>([&](auto I) {
        constexpr int cx = cx_of(I.value), cy = cy_of(I.value);
        d[I.value] = (double)S::load(emitted<NEQ, ST, I.value>(
            src, g, cx == 0 ? x : (cx > 0 ? xm : xp), cy == 0 ? y : (cy > 0 ? ym : yp), k));
      });
      return;
    }
  }
  const int64_t P = g.plane;
  const int64_t r0 = (int64_t)y * g.nx, rm = (int64_t)ym * g.nx, rp = (int64_t)yp * g.nx;
  d[0] = (double)S::load(src[0 * P + r0 + x]);
  d[1] = (double)S::load(src[1 * P + r0 + xm]);
  d[2] = (double)S::load(src[2 * P + rm + x]);
  d[3] = (double)S::load(src[3 * P + r0 + xp]);
  d[4] = (double)S::load(src[4 * P + rp + x]);
  d[5] = (double)S::load(src[5 * P + rm + xm]);
  d[6] = (double)S::load(src[6 * P + rm + xp]);
  d[7] = (double)S::load(src[7 * P + rp + xp]);
  d[8] = (double)S::load(src[8 * P + rp + xm]);
}

// rho - rho0 and j of shifted populations (sum w_i = 1, sum w_i c_i = 0).
__device__ __forceinline__ void moments64(const double (&d)[9], double& drho, double& jx,
                                          double& jy) {
  drho = d[0] + ((d[1] + d[3]) + (d[2] + d[4])) + ((d[5] + d[7]) + (d[6] + d[8]));
  jx = (d[1] - d[3]) + (d[5] - d[7]) + (d[8] - d[6]);
  jy = (d[2] - d[4]) + (d[5] - d[7]) + (d[6] - d[8]);
}

}  // namespace
}  // namespace oreg
