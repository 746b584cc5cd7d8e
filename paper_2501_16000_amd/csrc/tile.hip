// tile.hip -- the tile sweep: many time steps of a small D2Q9 lattice per
// launch, with the populations exchanged through LDS.
//
// One workgroup owns a region of at most 1024 nodes, one node per thread.  The
// first step pulls its populations from the source buffer, every further step
// from LDS, and the last one stores to the destination buffer.  Where a tile
// covers an axis of the lattice completely, that axis wraps inside LDS;
// otherwise the region carries a halo of L - 1 nodes on each side (the first
// step needs none, it reads memory), and each step computes one node less on
// every such side.
//
// What bounds it: latency.  These lattices hold a few wavefronts per CU, a
// launch costs about 2.5 us and a step the dependent chain of one collision,
// the LDS exchange and a barrier (0.37 us with one wavefront per SIMD), so the
// kernel runs many steps per launch and spreads every step over as many CUs
// as there are.  The strip pipeline runs a launch's steps one after the other
// in each wavefront (17 row steps of up to 7 collisions for 3 output rows).
// Measured, us per step, one sweep launch per step / strips / tiles: 128^2
// F64 3.26 / 2.46 / 1.03; 800 x 1 F64 2.59 / 2.23 / 0.45; 16384 x 4 F32S
// 2.81 / 4.02 / 0.68; 256^2 F32S 4.0 / 3.8 / 1.3.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dispatch.hpp"

namespace oreg {
namespace {
using namespace detail;

template <int EQ, int COLL, int BC, int ST>
__global__ __launch_bounds__(kTileNodes) void tile_kernel(
    const typename Storage<ST>::T* __restrict__ src, typename Storage<ST>::T* __restrict__ dst,
    Geometry g, Coef64 c, TileShape s, int L) {
  using S = Storage<ST>;
  using R = typename S::R;
  using T = typename S::T;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  T* const lds = reinterpret_cast<T*>(lds_raw);
  const int n = threadIdx.x;
  const int N = blockDim.x;  // nodes of one LDS plane
  const int rx = s.rx, ry = s.ry;
  const int ly = n / rx, lx = n - ly * rx;
  const int by = blockIdx.x / s.tx, bx = blockIdx.x - by * s.tx;
  // Column and row of the node, before the periodic wrap.
  const int X = bx * s.ox - s.hx + lx, Y = by * s.oy - s.hy + ly;
  int x = X, y = Y;
  if (x < 0) x += g.nx;
  if (x >= g.nx) x -= g.nx;
  if (y < 0) y += g.ny;
  if (y >= g.ny) y -= g.ny;
  // Steps this node can take: the distance to the nearest region edge that is
  // not a periodic wrap, plus one; 0 for threads past the region and for
  // columns and rows past the lattice's last tile (their images belong to
  // other tiles).
  int reach = ly < ry ? L : 0;
  if (s.hx > 0) reach = min(reach, min(lx, rx - 1 - lx) + 1);
  if (s.hy > 0) reach = min(reach, min(ly, ry - 1 - ly) + 1);
  if (X - s.hx >= g.nx || Y - s.hy >= g.ny) reach = 0;
  const bool owned = lx >= s.hx && lx < rx - s.hx && ly >= s.hy && ly < ry - s.hy && X < g.nx && Y < g.ny;
  const bool wall = BC == LB_BC_BOUNCEBACK && (x == 0 || x == g.nx - 1);
  const Coeffs<R> k(c);

  R f[9];
  auto update = [&]() {
    if (wall) {
      R r[9];
      unroll<0, 9>([&](auto I) { r[I.value] = f[opp_of(I.value)]; });
      unroll<0, 9>([&](auto I) { f[I.value] = r[I.value]; });
    } else {
      collide<EQ, COLL, S::shifted, S::delta_u>(f, k);
    }
  };
  // Population i >= 1 of the LDS buffer b lives in plane 8 b + i - 1; the rest
  // population stays with its thread (rounded through the storage format like
  // the others).
  auto publish = [&](int b) {
    T* const p = lds + b * 8 * N + n;
    unroll<1, 9>([&](auto I) { p[(I.value - 1) * N] = S::store(f[I.value]); });
    f[0] = S::load(S::store(f[0]));
  };

  if (reach > 0) {
    const int xm = wrap_dec(x, g.nx), xp = wrap_inc(x, g.nx);
    const int ym = wrap_dec(y, g.ny), yp = wrap_inc(y, g.ny);
    const int64_t P = g.plane;
    const int64_t r0 = (int64_t)y * g.nx, rm = (int64_t)ym * g.nx, rp = (int64_t)yp * g.nx;
    const T v[9] = {src[r0 + x],         src[P + r0 + xm],     src[2 * P + rm + x],
                    src[3 * P + r0 + xp], src[4 * P + rp + x],  src[5 * P + rm + xm],
                    src[6 * P + rm + xp], src[7 * P + rp + xp], src[8 * P + rp + xm]};
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = S::load(v[i]);
    update();
    if (L > 1) publish(0);
  }
  // LDS column and row neighbours (wrapped; only nodes whose neighbours are in
  // the region, or that wrap, use them).
  const int lxm = lx == 0 ? rx - 1 : lx - 1, lxp = lx == rx - 1 ? 0 : lx + 1;
  const int l0 = ly * rx, lm = (ly == 0 ? ry - 1 : ly - 1) * rx, lp = (ly == ry - 1 ? 0 : ly + 1) * rx;
  for (int t = 2; t <= L; ++t) {
    // Step t reads the buffer that step t - 1 wrote and writes the other one,
    // whose readers (step t - 1) are all past this barrier.
    __syncthreads();
    if (reach >= t) {
      const T* const p = lds + (t & 1) * 8 * N;
      f[1] = S::load(p[l0 + lxm]);
      f[2] = S::load(p[N + lm + lx]);
      f[3] = S::load(p[2 * N + l0 + lxp]);
      f[4] = S::load(p[3 * N + lp + lx]);
      f[5] = S::load(p[4 * N + lm + lxm]);
      f[6] = S::load(p[5 * N + lm + lxp]);
      f[7] = S::load(p[6 * N + lp + lxp]);
      f[8] = S::load(p[7 * N + lp + lxm]);
      update();
      if (t < L) publish((t & 1) ^ 1);
    }
  }
  if (owned) {
    T* const q = dst + (int64_t)y * g.nx + x;
#pragma unroll
    for (int i = 0; i < 9; ++i) q[i * g.plane] = S::store(f[i]);
  }
}

}  // namespace
using namespace detail;

hipError_t launch_tile_sweep(int eq, int coll, int bc, int st, const void* src, void* dst,
                             const Geometry& g, const Coef64& c, const TileShape& sh, int levels,
                             hipStream_t s) {
  const int nodes = sh.rx * sh.ry;
  if (levels < 1 || nodes < 1 || nodes > kTileNodes || g.nx > kTileMostSide || g.ny > kTileMostSide)
    return hipErrorInvalidValue;
  const int threads = (nodes + 63) / 64 * 64;
  return with_storage(st, [&](auto ST) {
    using T = typename Storage<ST.value>::T;
    const size_t lds = levels > 1 ? 2 * 8 * (size_t)threads * sizeof(T) : 0;
    return with_eq(eq, [&](auto EQ) {
      return with_coll(coll, [&](auto CO) {
        return with_bc(bc, [&](auto BC) {
          tile_kernel<EQ.value, CO.value, BC.value, ST.value>
              <<<(unsigned int)(sh.tx * sh.ty), threads, lds, s>>>(
                  static_cast<const T*>(src), static_cast<T*>(dst), g, c, sh, levels);
          return hipGetLastError();
        });
      });
    });
  });
}

}  // namespace oreg
