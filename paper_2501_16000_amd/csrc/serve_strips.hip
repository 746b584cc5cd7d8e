// serve_strips.hip -- the server's batched launch by column strips: the strip
// pipeline of fused_impl.hpp over the work items of every resident lattice (F64,
// and the 16-bit formats when the resident set is large).
#include "fused_impl.hpp"

namespace oreg {
namespace {

// Batched form of fused_sweep_kernel for the server: each wavefront takes one
// work item (lattice, column strip, row block) of a descriptor table and runs
// the same pipeline with that lattice's own step count kl <= KMAX and row
// block height.  Strips are KMAX-wide at every kl, so the item layout of a
// lattice does not change when its last launch has fewer steps.
template <int KMAX, int EQ, int ST>
__global__ __launch_bounds__(256) void batched_fused_kernel(const LatticeDesc* __restrict__ d,
                                                            const int* __restrict__ map,
                                                            int64_t items, int64_t T) {
  using S = Storage<ST>;
  using Tt = typename S::T;
  constexpr int W = 64 - 2 * KMAX;
  // The wavefront index is uniform: with readfirstlane the descriptor loads
  // become scalar loads and the lattice's parameters stay in scalar
  // registers (without it they took 26-30 VGPRs).
  const int64_t item =
      (int64_t)xcd_block() * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (item >= items) return;  // whole wavefronts leave together
  const LatticeDesc& L = d[map[item]];
  const int local = (int)(item - L.tile_begin);
  const int strip = local % L.strips, seg = local / L.strips;
  const int H = L.rows;
  const int64_t t = T - L.admit_T;
  const Tt* __restrict__ src = static_cast<const Tt*>(L.buf[t & 1]);
  Tt* __restrict__ dst = static_cast<Tt*>(L.buf[(t + 1) & 1]);
  const Coeffs<typename S::R> k(L.coef);
  // The step count is uniform over the wavefront: branch to the pipeline
  // compiled for it.
  unroll<1, KMAX + 1>([&](auto KL) {
    if (L.kl == KL.value)
      fused_strip<KL.value, KMAX, EQ, LB_COLL_OREG, LB_BC_PERIODIC, ST>(
          src, dst, L.nx, L.ny, L.plane, strip * W, seg * H, H, k, lane);
  });
}

}  // namespace

hipError_t launch_batched_fused(int eq, int st, const LatticeDesc* d, const int* item_map,
                                int64_t items, int64_t T, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  return with_eq(eq, [&](auto EQ) {
    auto go = [&](auto ST) {
      batched_fused_kernel<FusedLevels<ST.value>::K, EQ.value, ST.value>
          <<<(unsigned int)((items + 3) / 4), 256, 0, s>>>(d, item_map, items, T);
      return hipGetLastError();
    };
    if (st == LB_F64) return go(IC<LB_F64>{});
    if (st == LB_F16S) return go(IC<LB_F16S>{});
    if (st == LB_BF16S) return go(IC<LB_BF16S>{});
    return hipErrorInvalidValue;
  });
}

}  // namespace oreg
