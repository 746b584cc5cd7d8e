// march3.hip -- the D3Q27 OReg sweep on boxes stored as ten numbers per node
// instead of 27 populations.
//
// The OReg update keeps only rho, u and the six stress terms of a node
// (d3q27.hpp: reduce); its 27 post-collision populations are a function of
// those (emit).  A buffer of such a box therefore holds either the populations
// (after an init or a restored checkpoint) or, after a step, ten values per
// node in the collision's register type.  A device flag per buffer says which,
// so that the kernels, not the host, follow the state (a captured graph may
// be replayed after a new init).  The results are the same bit for bit: the
// populations are formed by the same operations on the same values, one
// launch later.
//
// One step: a workgroup marches a tile of columns along z.  For every plane it
// loads the ten numbers of the tile and one halo node around it (prefetched a
// plane ahead), forms the 27 populations, rounds them through the storage
// format and passes them through LDS; each output node gathers the 27 that
// stream to it, and keeps the six plane sums of each c_z group until the three
// planes that make up its moments have passed.
//
// What bounds it: HBM traffic in F64 (160 instead of 432 bytes per node and
// step; counters show 3.0 GB per 256^3 step, the reads 1.26 times the
// algorithmic ones), and in F32S the arithmetic of the halo nodes and the two
// phases of a plane, which share one workgroup per CU.  256^3, us per step,
// population sweep / march: F64 1322 / 552, F32S 648 / 352; 128^3: 195 / 83,
// 98 / 41.
//
// The same march reads rho and u (kMoments) and the sums of lb3_diagnostics
// (kSums) in one pass.  A step and diagnostics, with the sums from
// populations / written out for the purpose / formed here: 256^3 F64 1920 / 2099
// / 1039 us, F32S 978 / 1174 / 706; 64^3 F64 57 / 71 / 57.
#include <hip/hip_runtime.h>

#include "dispatch.hpp"
#include "kernels3.hpp"

namespace oreg {
namespace {
using namespace detail;

enum { kStep = 0, kMoments = 1, kSums = 2 };
constexpr int kNSums = 7;

// Cell (x, y, z) with one periodic wrap per axis.
__device__ __forceinline__ int wrap1(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

template <int EQ, int ST, int MODE>
__global__ __launch_bounds__(kMarchThreads) void march3_kernel(const void* __restrict__ src,
                                                           void* __restrict__ dst,
                                                           const unsigned int* __restrict__ fmt_src,
                                                           unsigned int* __restrict__ fmt_dst,
                                                           Geometry3 g, Coef64 c, double theta, MarchShape s) {
  using S = Storage<ST>;
  using R = typename S::R;
  using T = typename S::T;
  using A = typename std::conditional<MODE == kStep, R, double>::type;  // type of the sums
  constexpr int NR = kMarchRegion;
  // Two LDS buffers where they fit save the barrier between a plane's reads
  // and the next plane's writes (64 x 8 tiles, 256^3: F32S 405 -> 399 us).
  constexpr int BUFS = 2 * 27 * NR * (int)sizeof(T) <= 160 * 1024 ? 2 : 1;
  __shared__ T buffers[BUFS][27 * NR];
  const int tid = threadIdx.x;
  const int block = xcd_block();
  const int tiles = s.ntx * s.nty;
  const int chunk = block / tiles, tile = block - chunk * tiles;
  const int bty = tile / s.ntx, btx = tile - bty * s.ntx;
  const int X0 = btx * s.tx, Y0 = bty * s.ty, z0 = chunk * s.zc;
  const int z1 = min(z0 + s.zc, g.nz);
  const Coeffs<R> k(c);

  // Output node of this thread.
  const int oy = tid / s.tx, ox = tid - oy * s.tx;
  const bool out = tid < s.tx * s.ty && X0 + ox < g.nx && Y0 + oy < g.ny;
  const int64_t ocell = (int64_t)(Y0 + oy) * g.nx + (X0 + ox);
  const int64_t plane = (int64_t)g.nx * g.ny;
  [[maybe_unused]] auto store = [&](int z, A drho, const A(&j)[3], const A(&M)[6]) {
    const int64_t cell = z * plane + ocell;
    if constexpr (MODE == kMoments) {
      double* const q = static_cast<double*>(dst);
      const double rho = c.rho0 + drho;
      q[cell] = rho;
#pragma unroll
      for (int a = 0; a < 3; ++a) q[(a + 1) * g.cells + cell] = j[a] / rho;
    } else if constexpr (MODE == kStep) {
      R v[d3::kParams];
      d3::reduce<S::shifted>(drho, j, M, k, v);
      R* const q = static_cast<R*>(dst) + cell;
#pragma unroll
      for (int i = 0; i < d3::kParams; ++i) q[i * g.cells] = v[i];
    }
  };
  [[maybe_unused]] double acc[kNSums] = {0, 0, 0, 0, 0, 0, 0};
  // finite: whether the node's 27 populations are (kSums only).
  auto finish = [&](int z, const d3::PlaneSums<A>& m, const d3::PlaneSums<A>& o,
                    const d3::PlaneSums<A>& p, [[maybe_unused]] bool finite) {
    A drho, j[3], M[6];
    d3::combine(m, o, p, drho, j, M);
    if constexpr (MODE == kSums) {
      if (!finite) {
        acc[6] += 1.0;
        return;
      }
      const double rho = c.rho0 + drho;
      const double ke = 0.5 * (j[0] * j[0] + j[1] * j[1] + j[2] * j[2]) / rho;
      acc[0] += rho;
      acc[1] += j[0];
      acc[2] += j[1];
      acc[3] += j[2];
      acc[4] += ke;
      acc[5] += 1.5 * rho * theta + ke;
    } else {
      store(z, drho, j, M);
    }
  };
  // The workgroup's sums, in a fixed order, to dst[block].
  [[maybe_unused]] auto write_sums = [&] {
    __shared__ double part[kMarchThreads / 64][kNSums];
#pragma unroll
    for (int i = 0; i < kNSums; ++i) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) acc[i] += __shfl_down(acc[i], o, 64);
      if ((tid & 63) == 0) part[tid >> 6][i] = acc[i];
    }
    __syncthreads();
    if (tid < kNSums) {
      double v = part[0][tid];
      for (int w = 1; w < kMarchThreads / 64; ++w) v += part[w][tid];
      static_cast<double*>(dst)[block * kNSums + tid] = v;
    }
  };
  [[maybe_unused]] auto all_finite = [](const A (&a)[9]) {
    bool f = true;
    if constexpr (MODE == kSums) {
#pragma unroll
      for (int i = 0; i < 9; ++i) f = f && isfinite(a[i]);
    }
    return f;
  };
  if (MODE == kStep && block == 0 && tid == 0) *fmt_dst = 1;

  if (*fmt_src == 0) {
    // Populations: every output node pulls its 27.
    const T* const f = static_cast<const T*>(src);
    const int x = X0 + ox, y = Y0 + oy;
    const int xs[3] = {wrap1(x + 1, g.nx), x, wrap1(x - 1, g.nx)};  // by c_x + 1
    const int ys[3] = {wrap1(y + 1, g.ny), y, wrap1(y - 1, g.ny)};
    for (int z = z0; out && z < z1; ++z) {
      d3::PlaneSums<A> sums[3];
      bool finite = true;
#pragma unroll
      for (int cz = 0; cz < 3; ++cz) {
        const int zs = wrap1(z + 1 - cz, g.nz);
        A v[9];
#pragma unroll
        for (int i = 0; i < 9; ++i)
          v[i] = (A)S::load(f[(9 * cz + i) * g.cells + zs * plane + (int64_t)ys[i / 3] * g.nx + xs[i % 3]]);
        sums[cz] = d3::plane_sums(v);
        finite = finite && all_finite(v);
      }
      finish(z, sums[0], sums[1], sums[2], finite);
    }
    if constexpr (MODE == kSums) write_sums();
    return;
  }

  // Region node of this thread: the tile with one node more on every side.
  const int rx = s.tx + 2, region = rx * (s.ty + 2);
  const int ry = tid / rx, rxx = tid - ry * rx;
  const int X = X0 - 1 + rxx, Y = Y0 - 1 + ry;
  const bool in = tid < region && X <= g.nx && Y <= g.ny;
  const R* const q0 = static_cast<const R*>(src) + (in ? (int64_t)wrap1(Y, g.ny) * g.nx + wrap1(X, g.nx) : 0);
  const int at = in ? tid : 0;
  const int from = (oy + 1) * rx + ox + 1;  // the output node's place in the region

  R v[d3::kParams];
  auto fetch = [&](int p) {
    const R* const q = q0 + wrap1(p, g.nz) * plane;
    if (in) {
#pragma unroll
      for (int i = 0; i < d3::kParams; ++i) v[i] = q[i * g.cells];
    }
  };
#pragma unroll
  for (int i = 0; i < d3::kParams; ++i) v[i] = R(0);
  fetch(z0 - 1);
  d3::PlaneSums<A> up1{}, up2{}, mid{};  // c_z = +1 of planes p - 1 and p - 2, c_z = 0 of p - 1
  [[maybe_unused]] bool up1_finite = true, up2_finite = true, mid_finite = true;
  for (int p = z0 - 1; p <= z1; ++p) {
    R w[d3::kParams];
#pragma unroll
    for (int i = 0; i < d3::kParams; ++i) w[i] = v[i];
    if (p < z1) fetch(p + 1);
    T* const lds = buffers[(p - z0 + 1) & (BUFS - 1)];
    if (in) {
      T* const l = lds + at;
      d3::emit_each<EQ, S::shifted>(w, k, [&](auto I, R f) { l[I.value * NR] = S::store(f); },
                                    [] { __builtin_amdgcn_sched_barrier(0); });
    }
    __syncthreads();
    if (out) {
      auto group = [&](auto CZ, bool& finite) {
        A a[9];
        unroll<0, 9>([&](auto I) {
          constexpr int cx = I.value % 3 - 1, cy = I.value / 3 - 1;
          a[I.value] = (A)S::load(lds[(9 * CZ.value + I.value) * NR + from - cy * rx - cx]);
        });
        const d3::PlaneSums<A> sums = d3::plane_sums(a);
        finite = all_finite(a);
        __builtin_amdgcn_sched_barrier(0);
        return sums;
      };
      if (p > z0) {
        bool down_finite;
        const d3::PlaneSums<A> down = group(IC<0>{}, down_finite);
        finish(p - 1, down, mid, up2, down_finite && mid_finite && up2_finite);
      }
      up2 = up1;
      up2_finite = up1_finite;
      if (p < z1) {
        mid = group(IC<1>{}, mid_finite);
        up1 = group(IC<2>{}, up1_finite);
      }
    }
    if (BUFS == 1 && p < z1) __syncthreads();
  }
  if constexpr (MODE == kSums) write_sums();
}

// The populations of a buffer that holds ten numbers per node, into alt (left
// alone if the buffer holds populations).
template <int EQ, int ST>
__global__ __launch_bounds__(kThreads) void expand3_kernel(const void* __restrict__ src,
                                                           typename Storage<ST>::T* __restrict__ alt,
                                                           const unsigned int* __restrict__ fmt,
                                                           Geometry3 g, Coef64 c) {
  using S = Storage<ST>;
  using R = typename S::R;
  if (*fmt == 0) return;
  const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= g.cells) return;
  const Coeffs<R> k(c);
  R q[d3::kParams], f[27];
#pragma unroll
  for (int i = 0; i < d3::kParams; ++i) q[i] = static_cast<const R*>(src)[i * g.cells + idx];
  d3::emit<EQ, S::shifted>(q, k, f);
  unroll<0, 27>([&](auto I) { alt[I.value * g.cells + idx] = S::store(f[I.value]); });
}

template <int MODE>
hipError_t launch_march(int eq, int st, const void* src, void* dst, const unsigned int* fmt_src,
                        unsigned int* fmt_dst, const Geometry3& g, const Coef64& c,
                        double theta, const MarchShape& s, hipStream_t q) {
  if (!march_shape_ok(s, g.nx, g.ny, g.nz)) return hipErrorInvalidValue;
  const unsigned int blocks = (unsigned int)((int64_t)s.ntx * s.nty * s.nzc);
  return with_eq(eq, [&](auto EQ) {
    auto go = [&](auto ST) {
      march3_kernel<EQ.value, ST.value, MODE>
          <<<blocks, kMarchThreads, 0, q>>>(src, dst, fmt_src, fmt_dst, g, c, theta, s);
      return hipGetLastError();
    };
    if (st == LB_F64) return go(IC<LB_F64>{});
    if (st == LB_F32S) return go(IC<LB_F32S>{});
    return hipErrorInvalidValue;
  });
}

}  // namespace

hipError_t launch_march3(int eq, int st, const void* src, void* dst, const unsigned int* fmt_src,
                         unsigned int* fmt_dst, const Geometry3& g, const Coef64& c,
                         const MarchShape& s, hipStream_t q) {
  return launch_march<kStep>(eq, st, src, dst, fmt_src, fmt_dst, g, c, 0.0, s, q);
}

hipError_t launch_march3_moments(int eq, int st, const void* src, double* out,
                                 const unsigned int* fmt, const Geometry3& g, const Coef64& c,
                                 const MarchShape& s, hipStream_t q) {
  return launch_march<kMoments>(eq, st, src, out, fmt, nullptr, g, c, 0.0, s, q);
}

hipError_t launch_march3_sums(int eq, int st, const void* src, double* partials,
                              const unsigned int* fmt, const Geometry3& g, const Coef64& c,
                              double theta_energy, const MarchShape& s, hipStream_t q) {
  return launch_march<kSums>(eq, st, src, partials, fmt, nullptr, g, c, theta_energy, s, q);
}

hipError_t launch_expand3(int eq, int st, const void* src, void* alt, const unsigned int* fmt,
                          const Geometry3& g, const Coef64& c, hipStream_t s) {
  const unsigned int blocks = (unsigned int)((g.cells + kThreads - 1) / kThreads);
  return with_eq(eq, [&](auto EQ) {
    auto go = [&](auto ST) {
      using T = typename Storage<ST.value>::T;
      expand3_kernel<EQ.value, ST.value><<<blocks, kThreads, 0, s>>>(src, static_cast<T*>(alt), fmt, g, c);
      return hipGetLastError();
    };
    if (st == LB_F64) return go(IC<LB_F64>{});
    if (st == LB_F32S) return go(IC<LB_F32S>{});
    return hipErrorInvalidValue;
  });
}

}  // namespace oreg
