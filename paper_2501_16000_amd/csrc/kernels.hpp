// kernels.hpp -- host-side launchers of the D2Q9 OReg kernels (gfx950).
//
// Internal storage convention of a lattice buffer: plane i holds the
// post-collision, not yet streamed populations g_i, so that the observable
// pre-collision state of Eq. (7) is f_i(x, t) = g_i(x - c_i) (periodic).
// A sweep pulls g_i(x - c_i) from one buffer, collides, and stores g_i(x)
// into the other; streaming is the pull.  Shifted storage keeps g_i - w_i rho0.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "d2q9.hpp"
#include "plan.hpp"

namespace oreg {

struct Geometry {
  int nx, ny;
  int64_t plane;  // nx * ny
};

// Most workgroups of the diagnostics reduction.  How many there are, the reduction
// order and so the FP64 result depend only on the lattice's size and storage and on
// the format of its buffer, not on the device.
constexpr int kDiagBlocks = 1024;

// One time step: src -> dst.
hipError_t launch_sweep(int eq, int coll, int bc, int st, const void* src, void* dst,
                        const Geometry& g, const Coef64& c, hipStream_t s);

// Work-items (threads) of the single-step sweep launch for storage st on an
// nx x ny lattice: nodes per row rounded up to the workgroup's tile, times
// ny, divided by the nodes per thread.  HIP launches stay below 2^32.
int64_t sweep_work_items(int st, int nx, int ny);

// Time steps one fused launch advances for a storage format.
int fused_levels(int st);

// Whether strip launches of this configuration store the five numbers of a
// node (d2q9.hpp: Params) instead of its populations: periodic OReg in F64.  A
// device flag per buffer then says what it holds (0: populations, as after an
// init or a restored checkpoint, 1: five numbers); the kernels read and set the
// flags, so that captured launches follow the state.  The launchers below take
// null flags where every buffer holds populations.
bool fused_numbers(int coll, int bc, int st);

// Whether a fused launch of `levels` steps (1 .. fused_levels(st)) is
// compiled for this collision and boundary: the full count always, fewer
// steps for periodic OReg lattices, a single one where it stores numbers.
bool fused_levels_available(int coll, int bc, int st, int levels);

// `levels` time steps in one launch: src -> dst; each column strip (of one
// wavefront, or of a workgroup of four: `waves`, see plan_strips) produces
// `rows` (a multiple of 3) output rows.
hipError_t launch_fused_sweep(int eq, int coll, int bc, int st, const void* src, void* dst,
                              const Geometry& g, const Coef64& c, int waves, int rows, int levels,
                              const unsigned int* fmt_src, unsigned int* fmt_dst,
                              hipStream_t s);

// SIMDs of the current device and wavefronts of the `levels`-step fused sweep
// for storage st, with strips of `waves` wavefronts, that one SIMD holds at once
// (zeros if the query fails).
struct FusedShape {
  int simds;
  int waves_per_simd;
  double four;  // gain of four resident workgroups (fused_rows)
};
FusedShape fused_shape(int st, int waves, int levels);

// Modelled time of one K-step fused launch on an nx x ny lattice with H
// output rows per strip of `waves` wavefronts, in row-collision units of one
// wavefront.
double fused_cost(int waves, int nx, int ny, int H, const FusedShape& sh, int K);

// Output rows per strip (a multiple of 3) that minimise fused_cost.
int fused_rows(int waves, int nx, int ny, const FusedShape& sh, int levels);

// `levels` time steps in one launch of the tile sweep (tile.hip) or the block
// sweep (block.hip): src -> dst.
hipError_t launch_tile_sweep(int eq, int coll, int bc, int st, const void* src, void* dst,
                             const Geometry& g, const Coef64& c, const TileShape& sh, int levels,
                             hipStream_t s);
hipError_t launch_block_sweep(int eq, int coll, int bc, int st, const void* src, void* dst,
                              const Geometry& g, const Coef64& c, const BlockShape& b, int levels,
                              hipStream_t s);

// g from fields (device FP64 [ny][nx] each); counts invalid input nodes
// (non-finite value or rho <= 0) into *bad.
hipError_t launch_init(int eq, int st, const double* rho, const double* ux, const double* uy,
                       void* dst, const Geometry& g, const Coef64& c, unsigned int* bad,
                       unsigned int* fmt, hipStream_t s);

// Planes i .. i + count - 1 of g from fin[count][ny][nx], pre-collision FP64
// populations (device).  Called in plane order for all nine, it counts invalid
// nodes (a value that is not finite, or a sum that is not positive) into *bad;
// sum[ny][nx] is its workspace.
hipError_t launch_import_planes(int st, int i, int count, const double* fin, void* dst, double* sum,
                                unsigned int* bad, const Geometry& g, const Coef64& c,
                                hipStream_t s);

// Planes i .. i + count - 1 of the pre-collision FP64 populations (device) from g.
hipError_t launch_export_planes(int eq, int st, int i, int count, const void* src, double* fout,
                                const Geometry& g, const Coef64& c, const unsigned int* fmt,
                                hipStream_t s);

// rho, ux, uy of the pre-collision state into out[3][ny][nx] (device FP64).
hipError_t launch_moments(int eq, int st, const void* src, double* out, const Geometry& g,
                          const Coef64& c, const unsigned int* fmt, hipStream_t s);

// Diagnostics of the pre-collision state: partials[kDiagBlocks][6] scratch,
// out[6] result (device FP64).
hipError_t launch_diagnostics(int eq, int st, const void* src, double* partials, double* out,
                              const Geometry& g, const Coef64& c, double theta_energy,
                              const unsigned int* fmt, hipStream_t s);

// The two readers of lattices with format flags (readers_f64.hip); *blocks
// receives the number of partial rows (at most kDiagBlocks).
hipError_t launch_strip_moments(int eq, const void* src, double* out, const Geometry& g,
                                const Coef64& c, const unsigned int* fmt, hipStream_t s);
hipError_t launch_strip_diagnostics(int eq, const void* src, double* partials, int* blocks,
                                    const Geometry& g, const Coef64& c, double theta_energy,
                                    const unsigned int* fmt, hipStream_t s);

// y-average of rho(x): out[nx] (device FP64); partials holds nx * ny doubles
// at most.
hipError_t launch_profile(int eq, int st, const void* src, double* out, double* partials,
                          const Geometry& g, const Coef64& c, const unsigned int* fmt,
                          hipStream_t s);

// ------------------------------------------------------------ serving --
// One resident lattice of a server, as the batched sweep reads it.
struct LatticeDesc {
  void* buf[2];        // A/B population buffers
  double* fields;      // 3 * plane FP64: initial fields, later the result moments
  int nx, ny;
  int64_t plane;       // nx * ny
  int64_t admit_T;     // server launch counter at admission; the state is in
                       // buf[(T - admit_T) % 2] before launch T
  int64_t tile_begin;  // first work item of this lattice
  int kl;              // time steps this launch advances the lattice
  int rows, cols;      // output rows and columns of a work item
  int strips;          // work items side by side
  Coef64 coef;
};

// tile_map[b] = index of the lattice that owns work item b (after the
// descriptors are in device memory).
hipError_t launch_tile_map(const LatticeDesc* d, int n, int* tile_map, int64_t tiles,
                           hipStream_t s);

// Batched launches: up to fused_levels(st) steps per lattice per launch (d[i].kl
// each).  launch_batched_fused (F64, F16S, BF16S): one wavefront per work item,
// a column strip of fused_strip_width(st) columns x a row block.
// launch_batched_block (shifted formats): one workgroup of `waves` wavefronts
// of `rows` rows per work item, a tile of the block sweep.
int fused_strip_width(int st);
hipError_t launch_batched_fused(int eq, int st, const LatticeDesc* d, const int* item_map,
                                int64_t items, int64_t T, hipStream_t s);
hipError_t launch_batched_block(int eq, int st, const LatticeDesc* d, const int* item_map,
                                int64_t items, int64_t T, int waves, int rows, hipStream_t s);

// Plain streaming copy of bytes / 16 16-byte words (copy.hip).
hipError_t launch_copy(const void* src, void* dst, int64_t bytes, hipStream_t s);

}  // namespace oreg
