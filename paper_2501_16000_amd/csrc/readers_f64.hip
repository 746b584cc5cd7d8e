// readers_f64.hip -- moments and diagnostics of F64 lattices whose buffers may
// hold five numbers per node instead of populations.
//
// A reader needs the populations that stream to each node.  Forming them
// anew for every neighbour costs nine evaluations per node (4096^2 moments:
// 502 us); one level of the strip pipeline forms each node's populations once
// and hands them on through registers and lane shifts.
#include "fused_impl.hpp"
#include "readers.hpp"

namespace oreg {
namespace {

constexpr int kWidth = 62;  // columns of a one-level strip

// Runs visit(pulled populations, y) over the wavefront's strip in either format.
template <int EQ, class Visit>
__device__ __forceinline__ void visit_strip(const double* __restrict__ src, const Geometry& g,
                                            const Coeffs<double>& k, int wave, int strips, int H,
                                            bool numbers, int lane, Visit&& visit) {
  const int strip = wave % strips, seg = wave / strips;
  if (numbers)
    fused_strip<1, 1, EQ, LB_COLL_OREG, LB_BC_PERIODIC, LB_F64, 1, false, kNums, kVisit>(
        src, nullptr, g.nx, g.ny, g.plane, strip * kWidth, seg * H, H, k, lane, 0, visit);
  else
    fused_strip<1, 1, EQ, LB_COLL_OREG, LB_BC_PERIODIC, LB_F64, 1, false, kPops, kVisit>(
        src, nullptr, g.nx, g.ny, g.plane, strip * kWidth, seg * H, H, k, lane, 0, visit);
}

template <int EQ>
__global__ __launch_bounds__(256) void moments_strip_kernel(const double* __restrict__ src,
                                                            double* __restrict__ out, Geometry g,
                                                            Coef64 c, int strips, int items, int H,
                                                            const unsigned int* __restrict__ fmt) {
  if (*fmt == 0) {
    // Populations: every node for itself.  A strip's rows wait for each other
    // (1024^2: 21.0 us, 17.9 like this).
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < g.plane; idx += stride) {
      const int y = (int)(idx / g.nx);
      double d[9], rho, jx, jy;
      gather64<LB_F64, kPopsOnly>(src, g, (int)(idx - (int64_t)y * g.nx), y, c, false, d);
      moments64(d, rho, jx, jy);
      out[idx] = rho;
      out[g.plane + idx] = jx / rho;
      out[2 * g.plane + idx] = jy / rho;
    }
    return;
  }
  const int wave = xcd_block() * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (wave >= items) return;
  const int x = (wave % strips) * kWidth - 1 + lane;
  visit_strip<EQ>(src, g, Coeffs<double>(c), wave, strips, H, true, lane,
                  [&](const double (&d)[9], int y) {
                    double rho, jx, jy;
                    moments64(d, rho, jx, jy);
                    double* const q = out + (int64_t)y * g.nx + x;
                    q[0] = rho;
                    q[g.plane] = jx / rho;
                    q[2 * g.plane] = jy / rho;
                  });
}

// One row of six sums per workgroup (at most kDiagBlocks workgroups; a lattice
// of more strips than they have wavefronts takes several per wavefront).
template <int EQ>
__global__ __launch_bounds__(256) void diag_strip_kernel(const double* __restrict__ src,
                                                         double* __restrict__ partials, Geometry g,
                                                         Coef64 c, double theta, int strips,
                                                         int items, int H,
                                                         const unsigned int* __restrict__ fmt) {
  __shared__ double part[4][6];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = blockIdx.x * 4 + wv;
  const int lane = threadIdx.x & 63;
  double acc[6] = {0, 0, 0, 0, 0, 0};
  for (int w = wave; w < items; w += gridDim.x * 4)
    visit_strip<EQ>(src, g, Coeffs<double>(c), w, strips, H, *fmt != 0, lane,
                    [&](const double (&d)[9], int) {
                      bool finite = true;
#pragma unroll
                      for (int i = 0; i < 9; ++i) finite = finite && isfinite(d[i]);
                      if (!finite) {
                        acc[5] += 1.0;
                        return;
                      }
                      double rho, jx, jy;
                      moments64(d, rho, jx, jy);
                      const double ke = 0.5 * (jx * jx + jy * jy) / rho;
                      acc[0] += rho;
                      acc[1] += jx;
                      acc[2] += jy;
                      acc[3] += ke;
                      acc[4] += rho * theta + ke;
                    });
#pragma unroll
  for (int k = 0; k < 6; ++k) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc[k] += __shfl_down(acc[k], o, 64);
  }
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < 6; ++k) part[wv][k] = acc[k];
  }
  __syncthreads();
  if (threadIdx.x < 6)
    partials[blockIdx.x * 6 + threadIdx.x] =
        ((part[0][threadIdx.x] + part[1][threadIdx.x]) + part[2][threadIdx.x]) + part[3][threadIdx.x];
}

// Rows per strip (a multiple of 3) that give at most 4 * blocks strips.
int rows_for(const Geometry& g, int blocks) {
  const int strips = (g.nx + kWidth - 1) / kWidth;
  const int segs = 4 * blocks / strips > 1 ? 4 * blocks / strips : 1;
  const int rows = (g.ny + segs - 1) / segs;
  return (rows + 2) / 3 * 3;
}

}  // namespace

hipError_t launch_strip_moments(int eq, const void* src, double* out, const Geometry& g,
                                const Coef64& c, const unsigned int* fmt, hipStream_t s) {
  const int H = rows_for(g, 2048), strips = (g.nx + kWidth - 1) / kWidth;
  const int items = strips * ((g.ny + H - 1) / H);
  return with_eq(eq, [&](auto EQ) {
    moments_strip_kernel<EQ.value><<<(unsigned int)((items + 3) / 4), 256, 0, s>>>(
        static_cast<const double*>(src), out, g, c, strips, items, H, fmt);
    return hipGetLastError();
  });
}

hipError_t launch_strip_diagnostics(int eq, const void* src, double* partials, int* blocks,
                                    const Geometry& g, const Coef64& c, double theta_energy,
                                    const unsigned int* fmt, hipStream_t s) {
  const int H = rows_for(g, kDiagBlocks), strips = (g.nx + kWidth - 1) / kWidth;
  const int items = strips * ((g.ny + H - 1) / H);
  *blocks = items < 4 * kDiagBlocks ? (items + 3) / 4 : kDiagBlocks;
  return with_eq(eq, [&](auto EQ) {
    diag_strip_kernel<EQ.value><<<(unsigned int)*blocks, 256, 0, s>>>(
        static_cast<const double*>(src), partials, g, c, theta_energy, strips, items, H, fmt);
    return hipGetLastError();
  });
}

}  // namespace oreg
