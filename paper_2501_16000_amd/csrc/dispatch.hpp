// dispatch.hpp -- helpers shared by the D2Q9 kernel translation units
// (kernels.hip and the per-storage fused_*.hip): runtime-to-template
// dispatch, periodic index wrap, the XCD-aware workgroup order, and the shape
// of the fused multi-step sweep for each storage format.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.hpp"

namespace oreg {
namespace detail {

constexpr int kThreads = 256;

template <int V>
using IC = std::integral_constant<int, V>;

// ------------------------------------------------------------- dispatch --
template <class F>
hipError_t with_storage(int st, F&& f) {
  switch (st) {
    case LB_F64: return f(IC<LB_F64>{});
    case LB_F32S: return f(IC<LB_F32S>{});
    case LB_F16S: return f(IC<LB_F16S>{});
    case LB_BF16S: return f(IC<LB_BF16S>{});
    default: return hipErrorInvalidValue;
  }
}
template <class F>
hipError_t with_eq(int eq, F&& f) {
  switch (eq) {
    case LB_EQ_GUIDED: return f(IC<LB_EQ_GUIDED>{});
    case LB_EQ_POLY2: return f(IC<LB_EQ_POLY2>{});
    default: return hipErrorInvalidValue;
  }
}
template <class F>
hipError_t with_coll(int coll, F&& f) {
  switch (coll) {
    case LB_COLL_OREG: return f(IC<LB_COLL_OREG>{});
    case LB_COLL_BGK: return f(IC<LB_COLL_BGK>{});
    default: return hipErrorInvalidValue;
  }
}
template <class F>
hipError_t with_bc(int bc, F&& f) {
  switch (bc) {
    case LB_BC_PERIODIC: return f(IC<LB_BC_PERIODIC>{});
    case LB_BC_BOUNCEBACK: return f(IC<LB_BC_BOUNCEBACK>{});
    default: return hipErrorInvalidValue;
  }
}

__device__ __forceinline__ int wrap_dec(int v, int n) { return v == 0 ? n - 1 : v - 1; }
__device__ __forceinline__ int wrap_inc(int v, int n) { return v == n - 1 ? 0 : v + 1; }
// (v + d) mod n for 0 <= v < n and any small d.  The sum itself may not fit an
// int: sides go up to 2^31 - 1.
__host__ __device__ __forceinline__ int wrap_add(int v, int d, int n) {
  d %= n;
  if (d < 0) d += n;
  return v >= n - d ? v - (n - d) : v + d;
}
__device__ __forceinline__ int wrap_sub(int v, int c, int n) {
  return c == 0 ? v : (c > 0 ? wrap_dec(v, n) : wrap_inc(v, n));
}

// Workgroups go to the 8 XCDs of the chip round-robin (workgroup b to XCD
// b mod 8), and each XCD has its own L2.  xcd_block() renumbers them (a
// bijection on 0 .. gridDim.x - 1) so that every XCD takes one contiguous
// range: neighbouring tiles, which share cache lines at their edges, run on
// the same XCD.  Used by the fused sweeps, whose strips share 2K halo
// columns (their HBM reads fell from 1.27-1.62 to 1.16-1.19 times the
// algorithmic bytes).
__device__ __forceinline__ int xcd_block() {
  const int nwg = gridDim.x, b = blockIdx.x, xcd = b % 8, per = nwg / 8, extra = nwg % 8;
  return xcd * per + (xcd < extra ? xcd : extra) + b / 8;
}

// Fused launches per storage.  K: steps per launch.  FP64: seven.  Stored as
// five numbers per node, 4096^2 launches of 1 .. 7 steps take 317, 334, 323,
// 331, 401, 476 and 559 us: up to four steps the strips' memory traffic sets
// the time, beyond that each step adds the 80 us of its collisions, so five to
// seven steps cost the same per step (80 us; stored as populations, seven steps
// took 655 us); lb_step takes fewer than seven where that is faster.
// The FP32 formats are bound by their collisions at K = 6 (F32S 4096^2: 0.33 ms
// per launch) and keep six.
// NW: wavefronts per strip.  The 32- and 16-bit formats share one 256-column
// strip per workgroup, whose rows pass through LDS at every level: their
// sweeps are bound by VALU issue, and the LDS reads replace the lane shifts
// (F32S 116 -> 107 instructions per collision) while the halo is 2K of 256
// instead of 64 columns.  us per step, a wavefront per strip with shifts in
// the wavefront / two wavefronts / four / eight: 4096^2 F16S 57.2 / 54.0 /
// 50.8 / 56.7, BF16S 59.7 / 57.5 / 54.9 / 60.3, 8192^2 polynomial F16S 263 /
// 237 / 219 / 233; F32S (four, edges only through LDS: 58.0) 58.2 / 55.4 /
// 61.5.  Fewer wavefronts have more halo, more wait longer at each barrier.
// The 16-bit formats also have strips of one wavefront (NARROW), for lattices whose
// rows fill the wide ones badly (plan_strips).
// F64 has registers for two wavefronts per SIMD only, which the six or seven
// barriers of a row stop too often: 2048^2 21.8 / 36.8 / 28.1, 4096^2 80.3 /
// 84.1 / 77.5.
template <int ST> struct FusedLevels {
  static constexpr int K = ST == LB_F64 ? 7 : 6, NW = ST == LB_F64 ? 1 : 4;
  static constexpr bool NARROW = ST == LB_F16S || ST == LB_BF16S;
};

// Fused launches of fewer than FusedLevels<ST>::K steps (lb_step's remainder)
// are compiled for periodic OReg lattices, the configuration the benchmark
// and the server use; other configurations run a remainder as block launches.
constexpr bool short_fused(int coll, int bc) {
  return coll == LB_COLL_OREG && bc == LB_BC_PERIODIC;
}

// Whether strip launches store the five numbers of a node instead of its nine
// populations (fused_strip): periodic OReg in FP64, whose strips are bound by
// their memory traffic.  F32S strips are bound by VALU issue, and the 16-bit
// formats' nine populations (18 bytes) are smaller than five FP32 numbers.
constexpr bool stores_numbers(int coll, int bc, int st) {
  return short_fused(coll, bc) && st == LB_F64;
}

}  // namespace detail

// The fused sweeps of one storage format (fused_*.hip, one translation unit
// per format so that they compile in parallel).
template <int ST>
hipError_t fused_launch_st(int eq, int coll, int bc, const void* src, void* dst, const Geometry& g,
                           const Coef64& c, int waves, int rows, int levels,
                           const unsigned int* fmt_src, unsigned int* fmt_dst, hipStream_t s);
template <int ST>
hipError_t fused_occupancy_st(int waves, int levels, int* blocks);
}  // namespace oreg
