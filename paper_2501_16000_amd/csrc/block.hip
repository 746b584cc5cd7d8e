// block.hip -- the block sweep: several time steps of a D2Q9 lattice per
// launch, with a rectangle of the lattice held in the registers of one
// workgroup.
//
// A workgroup of W wavefronts owns 64 columns x (W RR) rows: lane l holds
// column l, wavefront w the rows w RR .. w RR + RR - 1, all nine populations
// of every row in registers.  The first step pulls from the source buffer, so
// L steps need a halo of L - 1 nodes on each side; each later step updates
// the rows in place, top down: the y neighbours are registers of the same
// lane, the x neighbours arrive by one-lane DPP shifts, and only the first
// and last row of every wavefront go through LDS (six values per lane and
// step, double buffered, one barrier per step).
//
// What bounds it: VALU issue.  A node update costs the collision plus the six
// lane shifts (in FP32 most of them fold into the consuming instruction), and
// on a 4096^2 F32S lattice the launch runs at 95 % of the issue rate of the
// row updates it does (L = 6, 8 x 8 rows: 64 x 64 nodes computed for 54 x 54
// stored).  Against a strip pipeline that marches down the lattice, the
// rectangle has no serial pipeline fill (2 L rows per strip), which is what
// small and middle lattices spent their time on.  Measured, us per step,
// strips / blocks: 777 x 523 F32S 6.6 / 2.9, F16S 4.7 / 3.0; 1024^2 F32S 11.3
// / 5.3; 512^2 F64 3.9 / 2.9.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dispatch.hpp"
#include "lanes.hpp"

namespace oreg {
namespace {
using namespace detail;

// What passes between wavefronts w - 1 and w through LDS, double buffered: pops
// 4, 7, 8 of the first row of w and pops 2, 5, 6 of the last row of w - 1.
template <typename R> struct Edge {
  R up[2][3][64], dn[2][3][64];
};
template <int RR, int EQ, int COLL, int BC, int ST>
__device__ __forceinline__ void block_tile(const typename Storage<ST>::T* __restrict__ src,
                                           typename Storage<ST>::T* __restrict__ dst, int nx,
                                           int ny, int64_t P,
                                           const Coeffs<typename Storage<ST>::R>& k, int X0,
                                           int Y0, int ox, int oy, int W, int L) {
  using S = Storage<ST>;
  using R = typename S::R;
  using T = typename S::T;
  static_assert((kBlockWaves + 1) * sizeof(Edge<R>) == block_lds(ST, kBlockWaves));
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  extern __shared__ double edges[];
  Edge<R>&top = reinterpret_cast<Edge<R>*>(edges)[wv], &bottom = (&top)[1];
  const int h = L - 1, RY = W * RR;
  const int x = wrap_add(X0, lane - h, nx);
  int y = wrap_add(Y0, wv * RR - h, ny);
  const bool wall = BC == LB_BC_BOUNCEBACK && (x == 0 || x == nx - 1);

  auto update = [&](R(&N)[9]) {
    if (wall) {
      R r[9];
      unroll<0, 9>([&](auto I) { r[I.value] = N[opp_of(I.value)]; });
      unroll<0, 9>([&](auto I) { N[I.value] = r[I.value]; });
    } else {
      collide<EQ, COLL, S::shifted, S::delta_u>(N, k);
    }
    // Between steps the populations are rounded through the storage format, so
    // that a launch equals L single steps bit for bit.
    S::round2(N[0], N[1]);
    S::round2(N[2], N[3]);
    S::round2(N[4], N[5]);
    S::round2(N[6], N[7]);
    N[8] = S::load(S::store(N[8]));
  };
  // Ordering point after each row: without it the compiler interleaves the
  // rows' collisions and runs out of registers.
  auto pin = [](R(&N)[9]) {
    __asm__ volatile("" : "+v"(N[0]), "+v"(N[1]), "+v"(N[2]), "+v"(N[3]), "+v"(N[4]), "+v"(N[5]),
                     "+v"(N[6]), "+v"(N[7]), "+v"(N[8]));
  };

  R f[RR][9];
  {
    const int xm = wrap_dec(x, nx), xp = wrap_inc(x, nx);
#pragma unroll
    for (int r = 0; r < RR; ++r) {
      const int ym = wrap_dec(y, ny), yp = wrap_inc(y, ny);
      const T* const p0 = src + (int64_t)y * nx;
      const T* const pm = src + (int64_t)ym * nx;
      const T* const pp = src + (int64_t)yp * nx;
      f[r][0] = S::load(p0[x]);
      f[r][1] = S::load(p0[P + xm]);
      f[r][2] = S::load(pm[2 * P + x]);
      f[r][3] = S::load(p0[3 * P + xp]);
      f[r][4] = S::load(pp[4 * P + x]);
      f[r][5] = S::load(pm[5 * P + xm]);
      f[r][6] = S::load(pm[6 * P + xp]);
      f[r][7] = S::load(pp[7 * P + xp]);
      f[r][8] = S::load(pp[8 * P + xm]);
      y = yp;
    }
  }
#pragma unroll
  for (int r = 0; r < RR; ++r) {
    // F16S: without this one periodic BGK of eight rows took 163 VGPRs, three
    // wavefronts per SIMD instead of four (105 with it).
    if constexpr (ST == LB_F16S) pin(f[r]);
    update(f[r]);
    pin(f[r]);
  }
  // The outermost rows of the region read what no wavefront wrote; it would only
  // feed halo rows that are no longer valid, which are left out below.
  for (int t = 2; t <= L; ++t) {
    const int b = t & 1;
    top.up[b][0][lane] = f[0][4];
    top.up[b][1][lane] = f[0][7];
    top.up[b][2][lane] = f[0][8];
    bottom.dn[b][0][lane] = f[RR - 1][2];
    bottom.dn[b][1][lane] = f[RR - 1][5];
    bottom.dn[b][2][lane] = f[RR - 1][6];
    // One barrier per step: buffer b is written again two steps later, after
    // the barrier that this step's readers reach next.
    __syncthreads();
    R a2 = top.dn[b][0][lane], a5 = top.dn[b][1][lane], a6 = top.dn[b][2][lane];
    const R b4 = bottom.up[b][0][lane], b7 = bottom.up[b][1][lane], b8 = bottom.up[b][2][lane];
#pragma unroll
    for (int r = 0; r < RR; ++r) {
      const int j = wv * RR + r;  // row of the region: valid after t steps in [t - 1, RY - t]
      const R o2 = f[r][2], o5 = f[r][5], o6 = f[r][6];
      if (j >= t - 1 && j <= RY - t) {
        constexpr int last = RR - 1;
        const int q = r < last ? r + 1 : last;
        R N[9];
        N[0] = f[r][0];
        N[1] = from_left(f[r][1]);
        N[2] = a2;
        N[3] = from_right(f[r][3]);
        N[4] = r < last ? f[q][4] : b4;
        N[5] = from_left(a5);
        N[6] = from_right(a6);
        N[7] = from_right(r < last ? f[q][7] : b7);
        N[8] = from_left(r < last ? f[q][8] : b8);
        update(N);
#pragma unroll
        for (int i = 0; i < 9; ++i) f[r][i] = N[i];
      }
      a2 = o2;
      a5 = o5;
      a6 = o6;
      pin(f[r]);
    }
  }
  if (lane >= h && lane < h + ox && lane - h < nx - X0) {
#pragma unroll
    for (int r = 0; r < RR; ++r) {
      const int j = wv * RR + r;
      if (j >= h && j < h + oy && j - h < ny - Y0) {
        T* const q = dst + (int64_t)(Y0 + (j - h)) * nx + (X0 + (lane - h));
#pragma unroll
        for (int i = 0; i < 9; ++i) q[i * P] = S::store(f[r][i]);
      }
    }
  }
}

template <int RR, int EQ, int COLL, int BC, int ST>
__global__ __launch_bounds__(64 * kBlockWaves) void block_kernel(
    const typename Storage<ST>::T* __restrict__ src, typename Storage<ST>::T* __restrict__ dst,
    Geometry g, Coef64 c, int tx, int ox, int oy, int L) {
  // Neighbouring tiles share halo nodes: xcd_block keeps them on one XCD's L2.
  const int tile = xcd_block();
  const int by = tile / tx, bx = tile - by * tx;
  const Coeffs<typename Storage<ST>::R> k(c);
  block_tile<RR, EQ, COLL, BC, ST>(src, dst, g.nx, g.ny, g.plane, k, bx * ox, by * oy, ox, oy,
                                   blockDim.x >> 6, L);
}

// The server's batched launch: each workgroup takes one tile of one resident
// lattice and advances it by that lattice's own step count kl.  The tiles are
// laid out for the most steps a launch takes, so a lattice's last launch, of
// fewer steps, has the same ones.
template <int RR, int EQ, int ST>
__global__ __launch_bounds__(64 * kBlockWaves) void batched_block_kernel(
    const LatticeDesc* __restrict__ d, const int* __restrict__ map, int64_t first, int64_t T) {
  using Tt = typename Storage<ST>::T;
  const int64_t item = first + xcd_block();
  const LatticeDesc& L = d[map[item]];
  const int local = (int)(item - L.tile_begin);
  const int by = local / L.strips, bx = local - by * L.strips;
  const int64_t t = T - L.admit_T;
  const Coeffs<typename Storage<ST>::R> k(L.coef);
  block_tile<RR, EQ, LB_COLL_OREG, LB_BC_PERIODIC, ST>(
      static_cast<const Tt*>(L.buf[t & 1]), static_cast<Tt*>(L.buf[(t + 1) & 1]), L.nx, L.ny,
      L.plane, k, bx * L.cols, by * L.rows, L.cols, L.rows, blockDim.x >> 6, L.kl);
}

}  // namespace
using namespace detail;

hipError_t launch_batched_block(int eq, int st, const LatticeDesc* d, const int* item_map,
                                int64_t items, int64_t T, int waves, int rows, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  if (waves < 1 || waves > kBlockWaves) return hipErrorInvalidValue;
  return with_eq(eq, [&](auto EQ) {
    auto go = [&](auto RR, auto ST) {
      // one launch, unless the items ask for 2^32 work-items or more
      const int64_t most = launch_items(64 * waves);
      for (int64_t first = 0; first < items; first += most) {
        batched_block_kernel<RR.value, EQ.value, ST.value>
            <<<(unsigned int)std::min(most, items - first), 64 * waves,
               block_lds(ST.value, waves), s>>>(d, item_map, first, T);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
      return hipSuccess;
    };
    auto rr = [&](auto ST) -> hipError_t {
      if (rows == block_rows_small(ST.value)) return go(IC<block_rows_small(ST.value)>{}, ST);
      if (rows == block_rows_big(ST.value)) return go(IC<block_rows_big(ST.value)>{}, ST);
      return hipErrorInvalidValue;
    };
    if (st == LB_F32S) return rr(IC<LB_F32S>{});
    if (st == LB_F16S) return rr(IC<LB_F16S>{});
    if (st == LB_BF16S) return rr(IC<LB_BF16S>{});
    return hipErrorInvalidValue;
  });
}

hipError_t launch_block_sweep(int eq, int coll, int bc, int st, const void* src, void* dst,
                              const Geometry& g, const Coef64& c, const BlockShape& b, int levels,
                              hipStream_t s) {
  const int h = levels - 1;
  if (levels < 1 || b.waves < 1 || b.waves > kBlockWaves || b.ox < 1 || b.oy < 1 ||
      b.ox + 2 * h > 64 || b.oy + 2 * h > b.waves * b.rows ||
      (int64_t)b.tx * b.ox < g.nx || (int64_t)b.ty * b.oy < g.ny)
    return hipErrorInvalidValue;
  return with_storage(st, [&](auto ST) {
    using T = typename Storage<ST.value>::T;
    return with_eq(eq, [&](auto EQ) {
      return with_coll(coll, [&](auto CO) {
        return with_bc(bc, [&](auto BC) -> hipError_t {
          auto go = [&](auto RR) {
            block_kernel<RR.value, EQ.value, CO.value, BC.value, ST.value>
                <<<(unsigned int)(b.tx * b.ty), 64 * b.waves,
                   block_lds(ST.value, b.waves), s>>>(
                    static_cast<const T*>(src), static_cast<T*>(dst), g, c, b.tx, b.ox, b.oy,
                    levels);
            return hipGetLastError();
          };
          if (b.rows == block_rows_small(ST.value)) return go(IC<block_rows_small(ST.value)>{});
          if (b.rows == block_rows_big(ST.value)) return go(IC<block_rows_big(ST.value)>{});
          return hipErrorInvalidValue;
        });
      });
    });
  });
}

}  // namespace oreg
