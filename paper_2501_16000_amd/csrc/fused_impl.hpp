// fused_impl.hpp -- the fused multi-step D2Q9 sweep (K time steps per
// launch, register-resident row pipeline) with its host launcher as templates
// over the storage format.  Included by fused_f64.hip, fused_f32s.hip,
// fused_f16s.hip and fused_bf16s.hip, which instantiate them for one format
// each, by serve_strips.hip (its batched form) and by readers_f64.hip.
#pragma once

#include "dispatch.hpp"
#include "lanes.hpp"

namespace oreg {
namespace {
using namespace detail;

// ------------------------------------------------ multi-step (fused) sweep --
// K time steps per launch.  A strip of 64 columns belongs to a wavefront (FP64,
// and the server's strips), or one of 256 to a workgroup (NW in FusedLevels),
// and is marched down H output rows; lane l holds column X0 - K + l.  The rows
// of time level 0 come from memory; level k + 1 of row y is computed from the
// last three rows of level k (a sliding window kept in registers).  The x
// neighbours' populations arrive by one-lane shifts (DPP, or ds_bpermute for
// window rows of the 16-bit formats) in a wavefront's strip and through LDS in
// a workgroup's.  Every level loses one column on each side, so the 64 - 2K
// (256 - 2K) middle columns of level K are stored.  The rows
// needed above and below the strip's H rows (K on each side) are recomputed
// by the neighbouring strips.  Between levels the populations are rounded
// through the storage format, so the result equals K single-step sweeps bit
// for bit.  The 2K pipeline-fill rows are unrolled, so that which levels
// produce is known at compile time, and the steady-state loop (three rows
// per trip) has no branches apart from the store predicate.  H is a runtime
// multiple of 3 chosen per lattice (fused_rows).

// One-lane shifts (from_left, from_right in lanes.hpp) through the LDS crossbar
// (ds_bpermute: no LDS memory, no VALU issue slot), for values that are needed a
// step after they are shifted: the latency is hidden and the VALU keeps its slots for the
// collision.  src_byte is 4 x the source lane (wrapped, so edge lanes read
// a value from the other edge; they are outside the valid region).
__device__ __forceinline__ float lane_perm(float v, int src_byte) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(src_byte, __float_as_int(v)));
}

// Access to element (plane i, row r, column col) of the source and
// destination population buffers.  Global form: a 64-bit address per plane
// and row.  Buffer form (BUF): one resource descriptor per buffer, the plane
// offset i * P in a scalar register and the 32-bit in-plane byte offset per
// lane, so no 64-bit address arithmetic per access (3-5 fewer VALU
// instructions per collision; measured 1-2 % faster on 4096^2 in every
// format).  The buffer form needs the buffer below 2 GiB (its byte offsets
// and the descriptor's record count are 32-bit); the hardware range check
// returns zero for, and drops, any access beyond it.
template <typename Tt, bool BUF>
struct PlaneIO {
  const Tt* __restrict__ src;
  Tt* __restrict__ dst;
  int64_t P;
  int nx;
  __device__ PlaneIO(const Tt* s, Tt* d, int64_t p, int n) : src(s), dst(d), P(p), nx(n) {}
  __device__ Tt load(int i, int r, int col) const { return src[i * P + (int64_t)r * nx + col]; }
  __device__ void store(int i, int r, int col, Tt v) const {
    dst[i * P + (int64_t)r * nx + col] = v;
  }
};
template <typename Tt>
struct PlaneIO<Tt, true> {
  static constexpr int kDword3 = 0x00020000;  // raw buffer access, gfx9 family
  __amdgpu_buffer_rsrc_t rs, rd;
  uint32_t plane_bytes;
  int nx;
  __device__ PlaneIO(const Tt* s, Tt* d, int64_t p, int n)
      : rs(__builtin_amdgcn_make_buffer_rsrc(const_cast<Tt*>(s), 0,
                                             (int)(9 * p * (int64_t)sizeof(Tt)), kDword3)),
        rd(__builtin_amdgcn_make_buffer_rsrc(d, 0, (int)(9 * p * (int64_t)sizeof(Tt)), kDword3)),
        plane_bytes((uint32_t)(p * (int64_t)sizeof(Tt))),
        nx(n) {}
  __device__ uint32_t off(int r, int col) const {
    return ((uint32_t)r * (uint32_t)nx + (uint32_t)col) * (uint32_t)sizeof(Tt);
  }
  __device__ Tt load(int i, int r, int col) const {
    const uint32_t o = off(r, col), so = (uint32_t)i * plane_bytes;
    if constexpr (sizeof(Tt) == 8)
      return __builtin_bit_cast(Tt, __builtin_amdgcn_raw_buffer_load_b64(rs, o, so, 0));
    else if constexpr (sizeof(Tt) == 4)
      return __builtin_bit_cast(Tt, __builtin_amdgcn_raw_buffer_load_b32(rs, o, so, 0));
    else
      return __builtin_bit_cast(Tt, __builtin_amdgcn_raw_buffer_load_b16(rs, o, so, 0));
  }
  __device__ void store(int i, int r, int col, Tt v) const {
    const uint32_t o = off(r, col), so = (uint32_t)i * plane_bytes;
    if constexpr (sizeof(Tt) == 8)
      __builtin_amdgcn_raw_buffer_store_b64(
          __builtin_bit_cast(unsigned int __attribute__((ext_vector_type(2))), v), rd, o, so, 0);
    else if constexpr (sizeof(Tt) == 4)
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), rd, o, so, 0);
    else
      __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), rd, o, so, 0);
  }
};

// Largest population buffer (both A/B halves use the same size) that the
// buffer form of PlaneIO addresses.
constexpr int64_t kBufferFormBytes = 0x7fffffff;

// One strip: K time steps over the rows Y0 .. Y0 + H - 1 of the columns
// X0 .. X0 + 64 NW - 1 - 2 KS.  Lane l of wavefront w holds column
// X0 - KS + 64 w + l; KS >= K is the strip's halo width, so strip columns
// KS .. 64 NW - 1 - KS are stored.  NW = 1: one wavefront per strip.  NW > 1
// (SHARE): the NW wavefronts of a workgroup sweep one strip together, and every
// lane takes its neighbours' populations from LDS: only the workgroup's outer
// edges carry a halo, and no VALU instruction is spent on a lane shift.
//
// IN, OUT: what a buffer holds.  kPops: the nine populations.  kNums: the five
// numbers of the OReg update (d2q9.hpp: Params), which the last level stores
// instead of the populations it would form from them, and from which the next
// launch forms them when a row arrives: the same arithmetic, one launch later,
// with 40 instead of 72 bytes per node read and written in FP64.  OUT = kVisit:
// nothing is stored; the last level hands the populations pulled to each of
// its rows to visit(N, y) instead.
enum { kPops = 0, kNums = 1, kVisit = 2 };
struct NoVisit {
  template <typename R>
  __device__ void operator()(const R (&)[9], int) const {}
};
template <int K, int KS, int EQ, int COLL, int BC, int ST, int NW = 1, bool BUF = false,
          int IN = kPops, int OUT = kPops, class Visit = NoVisit>
__device__ __forceinline__ void fused_strip(const typename Storage<ST>::T* __restrict__ src,
                                            typename Storage<ST>::T* __restrict__ dst, int nx,
                                            int ny, int64_t P, int X0, int Y0, int H,
                                            const Coeffs<typename Storage<ST>::R>& k, int lane,
                                            int wv = 0, Visit&& visit = Visit{}) {
  using S = Storage<ST>;
  using R = typename S::R;
  using Tt = typename S::T;
  constexpr bool SHARE = NW > 1;
  const int J = H + 2 * K;  // rows of level 0 read (H is a multiple of 3)
  const int cs = 64 * wv + lane;  // column within the strip, halo included
  const int col = wrap_add(X0, cs - KS, nx);
  const bool store_lane = cs >= KS && cs < 64 * NW - KS && cs - KS < nx - X0;
  const int left_byte = ((lane - 1) & 63) << 2, right_byte = ((lane + 1) & 63) << 2;
  // Window shifts of one wavefront's strip through ds_bpermute for the 16-bit
  // formats (measured 16 % faster for F16S and 7 % for BF16S).  F64 shifts by
  // DPP: with ds_bpermute 4096^2 takes 83.4 instead of 78.9 us per step, through
  // LDS as with SHARE 86.9.
  constexpr bool PERM = !SHARE && (ST == LB_F16S || ST == LB_BF16S);
  // A window population as stored (pre-shifted with PERM) and as pulled at
  // the gather (shifted there without PERM).
  auto enter = [&](R v, int src_byte) -> R {
    if constexpr (PERM) return lane_perm(v, src_byte);
    else return v;
  };
  auto pull_left = [&](R v) -> R {
    if constexpr (SHARE || PERM) return v;
    else return from_left(v);
  };
  auto pull_right = [&](R v) -> R {
    if constexpr (SHARE || PERM) return v;
    else return from_right(v);
  };
  const bool wall = BC == LB_BC_BOUNCEBACK && (col == 0 || col == nx - 1);
  // Window of level lv: row j of the level lives in slot j % 3 and holds
  // pops 0, 1, 2, 3, 5, 6 (pops 4, 7, 8 of a row are used as soon as it
  // arrives).  With three slots and the row loop unrolled by three, a new row
  // always goes to the slot of a row that is no longer read, so the slot
  // roles are compile-time constants and the window slides without register
  // moves.
  R Sl[K][3][6];
  // Exchange (SHARE): a row that arrives at a level goes through LDS, from
  // which every lane takes its neighbours' populations; x.l: 1, 5, 8 of the
  // column to the left, x.r: 3, 6, 7 of the one to the right.  Two exchanges in
  // a row use different buffers, so one barrier each suffices: a wavefront that
  // writes the buffer again has passed the barrier that the others reach after
  // their reads.
  struct Neighbours {
    R l[3], r[3];
  };
  constexpr int XP = 64 * NW;  // plane of an exchange buffer
  __shared__ R exchange[SHARE ? 3 * 6 * XP + 2 : 1];
  auto pass = [&](int buffer, const R(&v)[9], Neighbours& x) {
    if constexpr (SHARE) {
      R* const e = exchange + 1 + buffer * 6 * XP + cs;
      e[0] = v[1];
      e[XP] = v[5];
      e[2 * XP] = v[8];
      e[3 * XP] = v[3];
      e[4 * XP] = v[6];
      e[5 * XP] = v[7];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        x.l[i] = e[i * XP - 1];
        x.r[i] = e[(3 + i) * XP + 1];
      }
    }
  };
  const PlaneIO<Tt, BUF> io(src, dst, P, nx);
  int row = (Y0 - K) % ny;
  if (row < 0) row += ny;
  static_assert((IN == kPops && OUT != kNums) || (COLL == LB_COLL_OREG && BC == LB_BC_PERIODIC &&
                                                  std::is_same<Tt, R>::value),
                "five numbers: periodic OReg, stored in the collision's type");
  constexpr int NI = IN == kNums ? kParams : 9;
  constexpr int NO = OUT == kNums ? kParams : OUT == kVisit ? 1 : 9;
  Tt nb[3][NI];  // level-0 rows: row j is loaded into nb[j % 3] one row ahead
#pragma unroll
  for (int i = 0; i < NI; ++i) nb[0][i] = io.load(i, row, col);
  // Output row y is stored one step after it is computed, before that step's
  // prefetch: the wait for the prefetched row then covers only stores issued
  // a whole step earlier, never the ones just issued.  Plain stores, not
  // nontemporal ones: a strip's row piece shares its end cache lines with
  // the neighbouring strips (same XCD, same time), which the L2 then merges;
  // measured on 4096^2, nontemporal stores made the fused sweep 6 % (F64),
  // 4 % (F16S) and 2 % (BF16S) slower and the served FP64 stream 7 % slower
  // (F32S unchanged).  The single-step sweep keeps nontemporal stores (3-6 %
  // faster there).
  Tt pend[NO];
  auto store_row = [&](int dy) {  // row Y0 + dy
    if (OUT != kVisit && store_lane && dy >= 0 && dy < ny - Y0) {
#pragma unroll
      for (int i = 0; i < NO; ++i) io.store(i, Y0 + dy, col, pend[i]);
    }
  };

  // One row step: row j of level 0 arrives and the first NP levels (those
  // whose three source rows are complete, NP = min(K, j / 2)) produce a row
  // of the next level.  NP is a compile-time constant: the fill steps are
  // unrolled and the steady steps have NP = K.
  auto one_row = [&](int j, auto SLOT, auto NPROD) {
    constexpr int q = decltype(SLOT)::value;  // j % 3
    constexpr int qa = (q + 1) % 3;           // slot of row j - 2
    constexpr int qb = (q + 2) % 3;           // slot of row j - 1
    constexpr int NP = decltype(NPROD)::value;
    R C[9];
    // Keep the first use of the row that arrives here at this step: without
    // the ordering point the compiler hoists it into the previous step, right
    // behind the load, and the wavefront waits for memory.
    if constexpr (IN == kNums) {
      Params<R> p{nb[q][0], nb[q][1], nb[q][2], nb[q][3], nb[q][4]};
      __asm__ volatile("" : "+v"(p.drho), "+v"(p.ux), "+v"(p.uy), "+v"(p.ks), "+v"(p.kt));
      emit<EQ, S::shifted>(p, k, C);
    } else {
#pragma unroll
      for (int i = 0; i < 9; ++i) C[i] = S::load(nb[q][i]);
    }
    __asm__ volatile("" : "+v"(C[0]), "+v"(C[1]), "+v"(C[2]), "+v"(C[3]), "+v"(C[4]), "+v"(C[5]),
                     "+v"(C[6]), "+v"(C[7]), "+v"(C[8]));
    if constexpr (NP == K) store_row(j - 1 - 2 * K);  // the previous step's output row
    [[maybe_unused]] Neighbours x;
    pass(q * K % 3, C, x);
    // Prefetch the next row of level 0.  The last step reloads its own row
    // (a cache hit) instead of skipping the load: an unconditional load
    // leaves nothing of the old buffer alive.
    if (j + 1 < J) row = wrap_inc(row, ny);
#pragma unroll
    for (int i = 0; i < NI; ++i) nb[qa][i] = io.load(i, row, col);
#pragma unroll
    for (int lv = 0; lv < K; ++lv) {
      // Slot q held row j - 3 of the level, which is no longer read.  With
      // SHARE and PERM, pops 1, 3, 5 and 6 enter the window already shifted to
      // the lane that pulls them (they are read one and two steps later).
      Sl[lv][q][0] = C[0];
      Sl[lv][q][1] = SHARE ? x.l[0] : enter(C[1], left_byte);
      Sl[lv][q][2] = C[2];
      Sl[lv][q][3] = SHARE ? x.r[0] : enter(C[3], right_byte);
      Sl[lv][q][4] = SHARE ? x.l[1] : enter(C[5], left_byte);
      Sl[lv][q][5] = SHARE ? x.r[1] : enter(C[6], right_byte);
      if (lv >= NP) break;  // no rows of level lv + 1 yet
      R N[9];
      const R(&A)[6] = Sl[lv][qa];  // row j - 2 (pops 2, 5, 6 used)
      const R(&B)[6] = Sl[lv][qb];  // row j - 1 (pops 0, 1, 3 used)
      N[0] = B[0];
      N[2] = A[2];
      N[4] = C[4];
      N[1] = pull_left(B[1]);
      N[3] = pull_right(B[3]);
      N[5] = pull_left(A[4]);
      N[6] = pull_right(A[5]);
      N[7] = SHARE ? x.r[2] : from_right(C[7]);
      N[8] = SHARE ? x.l[2] : from_left(C[8]);
      if constexpr (OUT == kNums) {
        if (lv + 1 == K) {
          const Params<R> p = reduce<EQ>(node_moments<S::shifted, S::delta_u>(N, k), k);
          pend[0] = p.drho, pend[1] = p.ux, pend[2] = p.uy, pend[3] = p.ks, pend[4] = p.kt;
          break;
        }
      } else if constexpr (OUT == kVisit) {
        if (lv + 1 == K) {
          const int dy = j - 2 * K;
          if (store_lane && dy >= 0 && dy < ny - Y0) visit(N, Y0 + dy);
          break;
        }
      }
      if (wall) {
        R r[9];
        unroll<0, 9>([&](auto I) { r[I.value] = N[opp_of(I.value)]; });
        unroll<0, 9>([&](auto I) { N[I.value] = r[I.value]; });
      } else {
        collide<EQ, COLL, S::shifted, S::delta_u>(N, k);
      }
      if (lv + 1 == K) {
        if constexpr (OUT == kPops)
#pragma unroll
        for (int i = 0; i < 9; ++i) pend[i] = S::store(N[i]);  // output row Y0 + j - 2K
      } else {
#pragma unroll
        for (int i = 0; i < 9; ++i) C[i] = N[i];
        S::round2(C[0], C[1]);
        S::round2(C[2], C[3]);
        S::round2(C[4], C[5]);
        S::round2(C[6], C[7]);
        C[8] = S::load(S::store(C[8]));
        // Materialise the level's row here: without this ordering point the
        // compiler interleaves the collisions of the straight-line steady
        // loop and runs out of registers.
        __asm__ volatile("" : "+v"(C[0]), "+v"(C[1]), "+v"(C[2]), "+v"(C[3]), "+v"(C[4]),
                         "+v"(C[5]), "+v"(C[6]), "+v"(C[7]), "+v"(C[8]));
        pass((q * K + lv + 1) % 3, C, x);
      }
    }
    // The fill steps pass fewer rows, so the next step may use the same buffer.
    if constexpr (SHARE && NP < K) __syncthreads();
  };
  // Pipeline fill: rows 0 .. 2K - 1, level lv + 1 starting at row 2 (lv + 1).
  unroll<0, 2 * K>([&](auto JJ) { one_row(JJ.value, IC<JJ.value % 3>{}, IC<JJ.value / 2>{}); });
  // Steady state: every level produces a row per step.
  for (int j = 2 * K; j < J; j += 3) {
    one_row(j, IC<(2 * K) % 3>{}, IC<K>{});
    one_row(j + 1, IC<(2 * K + 1) % 3>{}, IC<K>{});
    one_row(j + 2, IC<(2 * K + 2) % 3>{}, IC<K>{});
  }
  store_row(J - 1 - 2 * K);
}

// fmt_src, fmt_dst: the format flags of the two buffers (0: populations, 1: five
// numbers) of lattices that store five numbers after a launch, else null.
template <int K, int EQ, int COLL, int BC, int ST, int NW, bool BUF = false, bool NUMS = false>
__global__ __launch_bounds__(256) void fused_sweep_kernel(
    const typename Storage<ST>::T* __restrict__ src, typename Storage<ST>::T* __restrict__ dst,
    Geometry g, Coef64 c, int strips, int items, int H, const unsigned int* __restrict__ fmt_src,
    unsigned int* __restrict__ fmt_dst) {
  constexpr int W = 64 * NW - 2 * K;
  // Neighbouring strips share their halo columns, which then come from the
  // XCD's L2 instead of HBM a second time.  The wavefront index is uniform:
  // keep it (and every row base derived from it) in scalar registers.
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const Coeffs<typename Storage<ST>::R> k(c);
  const int item = NW == 1 ? xcd_block() * 4 + wv : xcd_block();
  if (item >= items) return;  // whole wavefronts, with NW > 1 whole workgroups, leave together
  const int strip = item % strips, seg = item / strips;
  auto sweep = [&](auto IN, auto OUT) {
    fused_strip<K, K, EQ, COLL, BC, ST, NW, BUF, IN.value, OUT.value>(
        src, dst, g.nx, g.ny, g.plane, strip * W, seg * H, H, k, lane, NW == 1 ? 0 : wv);
  };
  if constexpr (NUMS) {
    if (item == 0 && threadIdx.x == 0) *fmt_dst = 1;
    // Uniform over the launch: the pipeline of the buffer's format.
    if (*fmt_src != 0) sweep(IC<kNums>{}, IC<kNums>{});
    else sweep(IC<kPops>{}, IC<kNums>{});
  } else {
    sweep(IC<kPops>{}, IC<kPops>{});
  }
}

// Runs f(wavefronts per strip) if strips of that many are compiled.
template <int ST, class F>
hipError_t with_strip_waves(int waves, F&& f) {
  if (waves == FusedLevels<ST>::NW) return f(IC<FusedLevels<ST>::NW>{});
  if constexpr (FusedLevels<ST>::NARROW) {
    if (waves == 1) return f(IC<1>{});
  }
  return hipErrorInvalidValue;
}

}  // namespace

template <int ST>
hipError_t fused_launch_st(int eq, int coll, int bc, const void* src, void* dst, const Geometry& g,
                           const Coef64& c, int waves, int rows, int levels,
                           const unsigned int* fmt_src, unsigned int* fmt_dst, hipStream_t s) {
  using T = typename Storage<ST>::T;
  constexpr int K = FusedLevels<ST>::K;
  return with_eq(eq, [&](auto EQ) {
    return with_coll(coll, [&](auto CO) {
      return with_bc(bc, [&](auto BC) -> hipError_t {
        // The buffer form of the plane access (PlaneIO) for the periodic OReg
        // sweeps, when the population buffer is below 2 GiB.
        constexpr bool buf_config = short_fused(CO.value, BC.value);
        constexpr bool nums = stores_numbers(CO.value, BC.value, ST);
        const bool buf = buf_config && 9 * g.plane * (int64_t)sizeof(T) <= kBufferFormBytes;
        auto go = [&](auto L, auto WAVES) -> hipError_t {
          constexpr int NW = WAVES.value, W = 64 * NW - 2 * L.value;
          const int strips = (g.nx + W - 1) / W;
          const int segs = (g.ny + rows - 1) / rows;
          const int items = strips * segs;
          const unsigned int nblocks = (unsigned int)(NW == 1 ? (items + 3) / 4 : items);
          if constexpr (buf_config) {
            if (buf) {
              fused_sweep_kernel<L.value, EQ.value, CO.value, BC.value, ST, NW, true, nums>
                  <<<nblocks, 256, 0, s>>>(static_cast<const T*>(src), static_cast<T*>(dst), g, c,
                                           strips, items, rows, fmt_src, fmt_dst);
              return hipGetLastError();
            }
          }
          fused_sweep_kernel<L.value, EQ.value, CO.value, BC.value, ST, NW, false, nums>
              <<<nblocks, 256, 0, s>>>(static_cast<const T*>(src), static_cast<T*>(dst), g, c,
                                       strips, items, rows, fmt_src, fmt_dst);
          return hipGetLastError();
        };
        if (nums && (!fmt_src || !fmt_dst)) return hipErrorInvalidValue;
        return with_strip_waves<ST>(waves, [&](auto WAVES) -> hipError_t {
          if (levels == K) return go(IC<K>{}, WAVES);
          hipError_t e = hipErrorInvalidValue;
          if constexpr (short_fused(CO.value, BC.value)) {
            unroll<nums ? 1 : 2, K>([&](auto L) {
              if (levels == L.value) e = go(L, WAVES);
            });
          }
          return e;
        });
      });
    });
  });
}

template <int ST>
hipError_t fused_occupancy_st(int waves, int levels, int* blocks) {
  constexpr bool nums = stores_numbers(LB_COLL_OREG, LB_BC_PERIODIC, ST);
  auto occ = [&](auto L, auto NW) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(
        blocks,
        reinterpret_cast<const void*>(&fused_sweep_kernel<L.value, LB_EQ_GUIDED, LB_COLL_OREG,
                                                          LB_BC_PERIODIC, ST, NW.value, false, nums>),
        256, 0);
  };
  return with_strip_waves<ST>(waves, [&](auto NW) {
    hipError_t e = hipErrorInvalidValue;
    unroll<nums ? 1 : 2, FusedLevels<ST>::K + 1>([&](auto L) {
      if (levels == L.value) e = occ(L, NW);
    });
    return e;
  });
}

}  // namespace oreg
