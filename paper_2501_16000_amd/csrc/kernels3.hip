// kernels3.hip -- D3Q27 kernels for gfx950 and their launchers.
//
// The sweep is one pass per time step: every node pulls its 27 populations
// from the upwind neighbours (periodic wrap), collides in registers
// (d3q27.hpp) and stores 27 post-collision populations.  Every element of
// the source is read by exactly one node, so the pass moves
// 2 * 27 * sizeof(storage) bytes per node and is bound by HBM bandwidth.
//
// Work split: one wavefront per 64-node segment of an x-row, four per
// workgroup.  A segment's (y, z) is uniform across the wavefront, so the 27
// source rows are scalar base addresses and each lane adds only its own
// column (x, x - 1 or x + 1 with the periodic wrap).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "kernels3.hpp"

namespace oreg {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

template <int V>
using IC = std::integral_constant<int, V>;

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

// (v - c) mod n for c in {-1, 0, 1} and 0 <= v < n.
__host__ __device__ __forceinline__ int wrap_sub(int v, int c, int n) {
  if (c == 0) return v;
  if (c > 0) return v == 0 ? n - 1 : v - 1;
  return v == n - 1 ? 0 : v + 1;
}

// ---------------------------------------------------------------- sweep --
// Most wavefronts per workgroup of the sweep, per storage (measured on 256^3:
// 8 for F64 and 16 for F32S beat 4 by 2 %; 4 is best for the 16-bit formats).
// Smaller boxes take fewer (sweep3_waves).
template <int ST> struct Sweep3Waves { static constexpr int N = 4; };
template <> struct Sweep3Waves<LB_F64> { static constexpr int N = 8; };
template <> struct Sweep3Waves<LB_F32S> { static constexpr int N = 16; };

// PACKED: a wavefront takes 64 consecutive nodes of the box instead of a segment
// of one x-row (sweep3_packed); mx, my: division by nx and ny (magic).  ORDERED:
// all loads before the first use (sweep3_ordered).
template <int EQ, int COLL, int ST, bool PACKED, bool ORDERED>
__global__ __launch_bounds__(64 * Sweep3Waves<ST>::N) void sweep3_kernel(
    const typename Storage<ST>::T* __restrict__ src, typename Storage<ST>::T* __restrict__ dst,
    Geometry3 g, Coef64 c, unsigned int nseg, unsigned int tasks, unsigned int mx,
    unsigned int my) {
  using S = Storage<ST>;
  using R = typename S::R;
  using T = typename S::T;
  const unsigned int task = blockIdx.x * (blockDim.x >> 6) +
                            (unsigned int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (task >= tasks) return;
  const int64_t P = g.cells;
  T raw[27];
  bool active;
  T* q;  // the node in plane 0 of dst
  if constexpr (PACKED) {
    const unsigned int nx = g.nx, ny = g.ny;
    const unsigned int first = task * 64u, row0 = first / nx, z0 = row0 / ny;
    // Node of this lane; past the end of the box, the box's first nodes.
    const unsigned int t = first - row0 * nx + (threadIdx.x & 63), dy = __umulhi(t, mx);
    const unsigned int u = row0 - z0 * ny + dy, dz = __umulhi(u, my);
    const int x = (int)(t - dy * nx), y = (int)(u - dz * ny);
    int z = (int)(z0 + dz);
    active = z < g.nz;
    if (!active) z = 0;
    // Byte offsets within a plane, 32 bits each: the plane's start is uniform.
    const unsigned int E = sizeof(T), row_bytes = nx * E, layer_bytes = ny * row_bytes;
    unsigned int xs[3], ys[3], zs[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      xs[a] = (unsigned int)wrap_sub(x, a - 1, g.nx) * E;
      ys[a] = (unsigned int)wrap_sub(y, a - 1, g.ny) * row_bytes;
      zs[a] = (unsigned int)wrap_sub(z, a - 1, g.nz) * layer_bytes;
    }
    unroll<0, 27>([&](auto I) {
      constexpr int vx = d3::cx(I.value), vy = d3::cy(I.value), vz = d3::cz(I.value);
      const char* const p = reinterpret_cast<const char*>(src + I.value * P);
      raw[I.value] = *reinterpret_cast<const T*>(p + (zs[vz + 1] + ys[vy + 1] + xs[vx + 1]));
    });
    q = reinterpret_cast<T*>(reinterpret_cast<char*>(dst) + (zs[1] + ys[1] + xs[1]));
  } else {
    const unsigned int row = task / nseg;
    const unsigned int seg = task - row * nseg;
    const int y = (int)(row % (unsigned int)g.ny);
    const int z = (int)(row / (unsigned int)g.ny);
    const unsigned int x = seg * 64u + (threadIdx.x & 63);
    active = x < (unsigned int)g.nx;
    const int xc = active ? (int)x : g.nx - 1;  // lanes past the row end load a valid node
    const int xm = xc == 0 ? g.nx - 1 : xc - 1;
    const int xp = xc == g.nx - 1 ? 0 : xc + 1;
    // Start of the source row of g_i(x - c_i) for each (c_y, c_z).
    int64_t rows[3][3];
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int a = 0; a < 3; ++a)
        rows[a][b] = ((int64_t)wrap_sub(z, b - 1, g.nz) * g.ny + wrap_sub(y, a - 1, g.ny)) * g.nx;
    unroll<0, 27>([&](auto I) {
      constexpr int vx = d3::cx(I.value), vy = d3::cy(I.value), vz = d3::cz(I.value);
      const T* p = src + I.value * P + rows[vy + 1][vz + 1];
      raw[I.value] = p[vx == 0 ? xc : (vx > 0 ? xm : xp)];
    });
    q = dst + rows[1][1] + x;
  }
  if constexpr (ORDERED) __builtin_amdgcn_sched_barrier(0);
  R f[27];
#pragma unroll
  for (int i = 0; i < 27; ++i) f[i] = S::load(raw[i]);
  const Coeffs<R> k(c);
  d3::collide<EQ, COLL, S::shifted>(f, k);
  if (active) {
    unroll<0, 27>([&](auto I) { __builtin_nontemporal_store(S::store(f[I.value]), q + I.value * P); });
  }
}

// ---------------------------------------------------------- per node --
struct Node {
  int x, y, z;
};
__device__ __forceinline__ Node node_of(int64_t idx, const Geometry3& g) {
  const int64_t r = idx / g.nx;
  Node n;
  n.x = (int)(idx - r * g.nx);
  n.y = (int)(r % g.ny);
  n.z = (int)(r / g.ny);
  return n;
}
__device__ __forceinline__ int64_t cell_of(int x, int y, int z, const Geometry3& g) {
  return ((int64_t)z * g.ny + y) * g.nx + x;
}
// Cell that holds g_i(x - c_i) for node n.
__device__ __forceinline__ int64_t upwind(const Node& n, int i, const Geometry3& g) {
  return cell_of(wrap_sub(n.x, d3::cx(i), g.nx), wrap_sub(n.y, d3::cy(i), g.ny),
                 wrap_sub(n.z, d3::cz(i), g.nz), g);
}

template <int EQ, int ST>
__global__ __launch_bounds__(kThreads) void init3_kernel(const double* __restrict__ rho,
                                                         const double* __restrict__ ux,
                                                         const double* __restrict__ uy,
                                                         const double* __restrict__ uz,
                                                         typename Storage<ST>::T* __restrict__ dst,
                                                         Geometry3 g, Coef64 c,
                                                         unsigned int* __restrict__ bad,
                                                         unsigned int* __restrict__ fmt) {
  using S = Storage<ST>;
  using R = typename S::R;
  const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= g.cells) return;
  if (fmt && idx == 0) *fmt = 0;  // the buffer holds populations
  double r = rho[idx];
  double u[3] = {ux[idx], uy[idx], uz[idx]};
  if (!(isfinite(r) && isfinite(u[0]) && isfinite(u[1]) && isfinite(u[2]) && r > 0.0)) {
    atomicAdd(bad, 1u);
    r = 1.0;
    u[0] = u[1] = u[2] = 0.0;
  }
  const double u2[3] = {u[0] * u[0], u[1] * u[1], u[2] * u[2]};
  const Coeffs<double> k(c);
  double feq[27], deq[27];
  d3::equilibrium<EQ, S::shifted>(S::shifted ? r - c.rho0 : r, r, u, u2, k, feq, deq);
  // f_i(x, 0) = f^eq_i(x) is stored as g_i(x - c_i).
  const Node n = node_of(idx, g);
  unroll<0, 27>([&](auto I) { dst[I.value * g.cells + upwind(n, I.value, g)] = S::store((R)deq[I.value]); });
}

// Plane i of pre-collision populations.  sum carries the sum of a node's
// populations from one plane to the next; bad counts values that are not finite
// and, with the last plane, nodes whose sum is not positive.
template <int ST>
__global__ __launch_bounds__(kThreads) void import3_kernel(int i, const double* __restrict__ fin,
                                                           typename Storage<ST>::T* __restrict__ dst,
                                                           double* __restrict__ sum,
                                                           unsigned int* __restrict__ bad,
                                                           Geometry3 g, Coef64 c) {
  using S = Storage<ST>;
  using R = typename S::R;
  const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= g.cells) return;
  const double v = fin[idx], rho = (i == 0 ? 0.0 : sum[idx]) + v;
  if (i < 26) sum[idx] = rho;
  if (!isfinite(v) || (i == 26 && !(rho > 0.0))) atomicAdd(bad, 1u);
  const double w = S::shifted ? d3::shift64(d3::cx(i), d3::cy(i), d3::cz(i), c) : 0.0;
  dst[i * g.cells + upwind(node_of(idx, g), i, g)] = S::store((R)(v - w));
}

template <int ST>
__global__ __launch_bounds__(kThreads) void export3_kernel(int i,
                                                           const typename Storage<ST>::T* __restrict__ src,
                                                           const typename Storage<ST>::T* __restrict__ alt,
                                                           const unsigned int* __restrict__ fmt,
                                                           double* __restrict__ fout, Geometry3 g,
                                                           Coef64 c) {
  using S = Storage<ST>;
  if (fmt && *fmt != 0) src = alt;  // see launch_expand3
  const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= g.cells) return;
  const double w = S::shifted ? d3::shift64(d3::cx(i), d3::cy(i), d3::cz(i), c) : 0.0;
  fout[idx] = (double)S::load(src[i * g.cells + upwind(node_of(idx, g), i, g)]) + w;
}

// Pre-collision populations of a node in FP64, still shifted by w_i rho0.
template <int ST>
__device__ __forceinline__ void gather3(const typename Storage<ST>::T* __restrict__ src,
                                        const Geometry3& g, const Node& n, double (&d)[27]) {
  using S = Storage<ST>;
  unroll<0, 27>([&](auto I) { d[I.value] = (double)S::load(src[I.value * g.cells + upwind(n, I.value, g)]); });
}

template <int ST>
__global__ __launch_bounds__(kThreads) void moments3_kernel(const typename Storage<ST>::T* __restrict__ src,
                                                            double* __restrict__ out, Geometry3 g,
                                                            Coef64 c) {
  const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= g.cells) return;
  double d[27], drho, j[3], M[6];
  gather3<ST>(src, g, node_of(idx, g), d);
  d3::moments(d, drho, j, M);
  const double rho = c.rho0 + drho;
  out[idx] = rho;
#pragma unroll
  for (int a = 0; a < 3; ++a) out[(a + 1) * g.cells + idx] = j[a] / rho;
}

// ---------------------------------------------------------- diagnostics --
constexpr int kSums = 7;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  return v;
}

// Fixed-order block sum; result valid in thread 0.
__device__ __forceinline__ void block_sum(double (&v)[kSums]) {
  __shared__ double part[kWaves][kSums];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < kSums; ++k) v[k] = wave_sum(v[k]);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < kSums; ++k) part[wave][k] = v[k];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < kSums; ++k) {
      double s = part[0][k];
      for (int w = 1; w < kWaves; ++w) s += part[w][k];
      v[k] = s;
    }
  }
}

template <int ST>
__global__ __launch_bounds__(kThreads) void diag3_kernel(const typename Storage<ST>::T* __restrict__ src,
                                                         double* __restrict__ partials, Geometry3 g,
                                                         Coef64 c, double theta) {
  double acc[kSums] = {0, 0, 0, 0, 0, 0, 0};
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x; idx < g.cells; idx += stride) {
    double d[27], drho, j[3], M[6];
    gather3<ST>(src, g, node_of(idx, g), d);
    bool finite = true;
#pragma unroll
    for (int i = 0; i < 27; ++i) finite = finite && isfinite(d[i]);
    if (!finite) {
      acc[6] += 1.0;
      continue;
    }
    d3::moments(d, drho, j, M);
    const double rho = c.rho0 + drho;
    const double ke = 0.5 * (j[0] * j[0] + j[1] * j[1] + j[2] * j[2]) / rho;
    acc[0] += rho;
    acc[1] += j[0];
    acc[2] += j[1];
    acc[3] += j[2];
    acc[4] += ke;
    acc[5] += 1.5 * rho * theta + ke;
  }
  block_sum(acc);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < kSums; ++k) partials[blockIdx.x * kSums + k] = acc[k];
  }
}

__global__ __launch_bounds__(kThreads) void diag3_final_kernel(const double* __restrict__ partials,
                                                               int nblocks, double* __restrict__ out) {
  double acc[kSums] = {0, 0, 0, 0, 0, 0, 0};
  for (int b = threadIdx.x; b < nblocks; b += kThreads) {
#pragma unroll
    for (int k = 0; k < kSums; ++k) acc[k] += partials[b * kSums + k];
  }
  block_sum(acc);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < kSums; ++k) out[k] = acc[k];
  }
}

unsigned int blocks_for(int64_t n) { return (unsigned int)((n + kThreads - 1) / kThreads); }

}  // namespace

// ------------------------------------------------------------ launchers --
int64_t sweep3_tasks(const Geometry3& g) {
  return ((int64_t)g.nx + 63) / 64 * g.ny * g.nz;
}

// F64 rows that take one round of wavefronts, two per SIMD (2048), but more than
// one per SIMD.  They run fastest in workgroups of eight, one per CU, and with the
// loads left to the compiler: us per step, four and ordered : eight and free, 41^3
// 9.8 : 9.2, 45^3 10.8 : 9.5, 64 x 32 x 48 10.6 : 8.8, 100 x 30 x 25 10.3 : 8.6.
bool sweep3_one_round(const Geometry3& g, int elem) {
  return elem == 8 && sweep3_tasks(g) > 1024 && sweep3_tasks(g) <= 2048;
}

// Wavefronts per workgroup.  Other boxes of less than 8 M nodes run faster with
// four, which spread small boxes over more CUs (us per step, F64 eight / four:
// 32^3 6.9 / 5.6, 128^3 189 / 173; F32S sixteen / four: 32^3 7.8 / 4.3, 128^3
// 98 / 87).
unsigned int sweep3_waves(const Geometry3& g, unsigned int most, bool one_round) {
  return !one_round && g.cells < (8 << 20) ? std::min(4u, most) : most;
}

// Whether all 27 loads of a node come before their first use.  Left to itself the
// compiler pairs every F16S load with its conversion and waits for each in turn
// (64^3 16.4 us per step, ordered 7.7).  F64 has no conversions: ordered loads
// help only where each SIMD has one wavefront at most (free : ordered, 16^3 5.6 :
// 4.5, 64 x 32 x 30 6.7 : 5.4; 64 x 64 x 40 15.0 : 16.1, 128^3 182 : 179, 256^3
// 1319 : 1373).
bool sweep3_ordered(const Geometry3& g, int elem, bool packed) {
  return packed || elem < 8 || sweep3_tasks(g) <= 1024;
}

// Whether the sweep packs 64 consecutive nodes of the box into a wavefront.  A
// segment of a row leaves 64 ceil(nx / 64) - nx lanes idle and starts its lines
// unaligned; packed nodes cost 33 more instructions (of 577 in the 16-bit
// formats) for their addresses.  us per step of three boxes in flight, rows :
// packed: BF16S 17 x 28 x 200 6.8 : 3.6, 60^3 6.2 : 5.2, 100 x 84 x 60 15.0 :
// 11.6, 200 x 180 x 160 220 : 124, and with whole segments 128^3 43.7 : 44.5; F64
// BGK 150^3 357 : 290.  Boxes of too few wavefronts run faster spread over more
// of them (32^3 F64 3.5 : 4.0, 48 x 40 x 30 5.8 : 5.2; 169 x 20 x 16, 12 % idle,
// one step and moments 10.6 : 10.8), and so do F64 boxes of more nodes than one
// packed wavefront per SIMD holds (1024 of them) whose rows take one round (40^3
// 8.9 : 8.4 but 41^3 9.2 : 10.5, 43^3 9.3 : 10.4, 45^3 9.5 : 11.4, 100 x 30 x 25
// 8.6 : 10.1, 250 x 18 x 18 9.8 : 11.2; 46^3 11.9 : 11.2).  Addresses are 32-bit byte
// offsets, and __umulhi by ceil(2^32 / n) divides exactly below 2^32 / n.
bool sweep3_packed(const Geometry3& g, int elem) {
  if (g.cells > 65536 && sweep3_one_round(g, elem)) return false;
  return g.nx > 1 && g.ny > 1 && g.ny < 65000 && g.cells >= 45000 &&
         g.cells * elem < 4294967296LL &&
         (g.cells < 100000 ? 1.25 : 1.04) * (double)g.cells < 64.0 * (double)sweep3_tasks(g);
}

hipError_t launch_sweep3(int eq, int coll, int st, const void* src, void* dst, const Geometry3& g,
                         const Coef64& c, hipStream_t s) {
  const unsigned int nseg = ((unsigned int)g.nx + 63) / 64;
  auto magic = [](int n) { return (unsigned int)((4294967296ULL + n - 1) / (unsigned int)n); };
  return with_storage(st, [&](auto ST) {
    using T = typename Storage<ST.value>::T;
    constexpr int E = (int)sizeof(T);
    const bool packed = sweep3_packed(g, E), ordered = sweep3_ordered(g, E, packed);
    const unsigned int W =
        sweep3_waves(g, Sweep3Waves<ST.value>::N, !packed && sweep3_one_round(g, E));
    const unsigned int tasks = (unsigned int)(packed ? (g.cells + 63) / 64 : sweep3_tasks(g));
    const unsigned int nblocks = (tasks + W - 1) / W;
    return with_eq(eq, [&](auto EQ) {
      return with_coll(coll, [&](auto CO) {
        auto go = [&](auto PACKED, auto ORDERED) {
          sweep3_kernel<EQ.value, CO.value, ST.value, PACKED.value, ORDERED.value>
              <<<nblocks, 64 * W, 0, s>>>(static_cast<const T*>(src), static_cast<T*>(dst), g, c,
                                          nseg, tasks, magic(g.nx), magic(g.ny));
          return hipGetLastError();
        };
        if constexpr (E == 8)
          if (!ordered) return go(IC<0>{}, IC<0>{});
        return packed ? go(IC<1>{}, IC<1>{}) : go(IC<0>{}, IC<1>{});
      });
    });
  });
}

hipError_t launch_init3(int eq, int st, const double* rho, const double* ux, const double* uy,
                        const double* uz, void* dst, const Geometry3& g, const Coef64& c,
                        unsigned int* bad, unsigned int* fmt, hipStream_t s) {
  return with_storage(st, [&](auto ST) {
    using T = typename Storage<ST.value>::T;
    return with_eq(eq, [&](auto EQ) {
      init3_kernel<EQ.value, ST.value><<<blocks_for(g.cells), kThreads, 0, s>>>(
          rho, ux, uy, uz, static_cast<T*>(dst), g, c, bad, fmt);
      return hipGetLastError();
    });
  });
}

hipError_t launch_import3(int st, int i, const double* fin, void* dst, double* sum,
                          unsigned int* bad, const Geometry3& g, const Coef64& c, hipStream_t s) {
  return with_storage(st, [&](auto ST) {
    using T = typename Storage<ST.value>::T;
    import3_kernel<ST.value><<<blocks_for(g.cells), kThreads, 0, s>>>(i, fin, static_cast<T*>(dst),
                                                                      sum, bad, g, c);
    return hipGetLastError();
  });
}

hipError_t launch_export3(int st, int i, const void* src, const void* alt,
                          const unsigned int* fmt, double* fout, const Geometry3& g,
                          const Coef64& c, hipStream_t s) {
  return with_storage(st, [&](auto ST) {
    using T = typename Storage<ST.value>::T;
    export3_kernel<ST.value><<<blocks_for(g.cells), kThreads, 0, s>>>(
        i, static_cast<const T*>(src), static_cast<const T*>(alt), fmt, fout, g, c);
    return hipGetLastError();
  });
}

hipError_t launch_moments3(int st, const void* src, double* out, const Geometry3& g,
                           const Coef64& c, hipStream_t s) {
  return with_storage(st, [&](auto ST) {
    using T = typename Storage<ST.value>::T;
    moments3_kernel<ST.value><<<blocks_for(g.cells), kThreads, 0, s>>>(static_cast<const T*>(src),
                                                                        out, g, c);
    return hipGetLastError();
  });
}

hipError_t launch_diagnostics3_final(const double* partials, int n, double* out, hipStream_t s) {
  diag3_final_kernel<<<1, kThreads, 0, s>>>(partials, n, out);
  return hipGetLastError();
}

hipError_t launch_diagnostics3(int st, const void* src, double* partials, double* out,
                               const Geometry3& g, const Coef64& c, double theta_energy,
                               hipStream_t s) {
  return with_storage(st, [&](auto ST) {
    using T = typename Storage<ST.value>::T;
    diag3_kernel<ST.value><<<kDiag3Blocks, kThreads, 0, s>>>(static_cast<const T*>(src), partials,
                                                             g, c, theta_energy);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_diagnostics3_final(partials, kDiag3Blocks, out, s);
  });
}

}  // namespace oreg
