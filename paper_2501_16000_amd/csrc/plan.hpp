// plan.hpp -- which multi-step kernel advances a lattice, and with which
// shape: the launch model of the tile sweep (tile.hip) and the block sweep
// (block.hip), in plain host code.
//
// Both kernels advance a lattice L time steps per launch and recompute a halo
// around each tile, so a longer launch spends less on launches and memory and
// more on halos.  The choice minimises the modelled time per step; every
// choice gives the same populations bit for bit.
//
// The models were fitted to 33,000 timed launches (24 lattices from 32^2 and
// 800 x 1 to 3000^2, F64, F32S and F16S, every shape below): the chosen shape
// ran within 5 % of the fastest one on three lattices out of four, and within
// 26 % on the worst.  Times are microseconds.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "oreg.h"

namespace oreg {

// Tile sweep: the lattice in tx x ty tiles of ox x oy output nodes; a tile's
// region is rx x ry nodes (one per thread), with hx and hy halo nodes per
// side (levels - 1, or 0 on an axis that one tile covers and that wraps).
constexpr int kTileNodes = 1024;
constexpr int kTileMostSide = 2147483647 - 2 * kTileNodes;  // a tile past the end still fits an int
struct TileShape {
  int tx, ty;
  int ox, oy;
  int rx, ry;
  int hx, hy;
};

// Block sweep: the lattice in tx x ty tiles of ox x oy output nodes, each
// advanced by a workgroup of `waves` wavefronts that holds 64 columns x waves
// * rows rows in registers (halo: levels - 1 on every side).
constexpr int kBlockWaves = 8;
struct BlockShape {
  int tx, ty;
  int ox, oy;
  int waves, rows;
};

// Rows per wavefront of the block sweep, two sizes per storage: eight rows of
// nine populations take 197 - 250 VGPRs in F64 (two wavefronts per SIMD) and 105 -
// 111 in F32S and F16S (four); in BF16S eight rows do not fit four wavefronts
// per SIMD, six do.
constexpr int block_rows_small(int) { return 4; }
constexpr int block_rows_big(int st) { return st == LB_BF16S ? 6 : 8; }
// Wavefronts of the block sweep that one SIMD holds (from its VGPRs; polynomial
// OReg in four rows of 32-bit arithmetic holds six).
constexpr int block_waves_per_simd(int st, int rows) {
  return st == LB_F64 ? (rows == 4 ? 3 : 2) : (rows == 4 ? 7 : 4);
}
// LDS of one of its workgroups: what passes between its wavefronts (and both ends),
// twelve rows of 64 values.
constexpr int block_lds(int st, int waves) {
  return (waves + 1) * 12 * 64 * (st == LB_F64 ? 8 : 4);
}
// Workgroups of it that one CU holds.
constexpr int block_fit(int st, int rows, int waves) {
  return std::max(1, std::min(4 * block_waves_per_simd(st, rows) / waves,
                              160 * 1024 / block_lds(st, waves)));
}

enum class StepKind { sweep, tile, block };
constexpr int kPlanLevels = 128;  // most steps of one launch

struct StepPlan {
  StepKind kind = StepKind::sweep;
  int levels = 1;       // steps per launch
  double us = 0;        // modelled time of the launch
  TileShape tile{};
  BlockShape block{};
};

// Workgroups of `threads` that one HIP launch can have: fewer than 2^32 work-items.
constexpr int64_t launch_items(int threads) { return (int64_t)4294967295LL / threads; }

namespace plan_detail {

constexpr int kBytes[4] = {8, 4, 2, 2};

inline int div_up(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

inline bool one_launch(int tx, int ty, int threads) {
  return (int64_t)tx * ty <= launch_items(threads);
}

// Tile sweep.  Launch t0 + t1, a step `lat` plus `c` for every wavefront of
// the fullest SIMD that still has nodes to update, and 1/seg for every row
// segment the first step loads.
struct TileFit {
  double t0, lat, c, t1, seg;
};
constexpr TileFit kTileFit[4] = {{1.64, 0.040, 0.230, 1.71, 28.1},
                                 {3.30, 0.096, 0.175, 0.0, 41.1},
                                 {3.28, 0.146, 0.182, 0.0, 55.4},
                                 {3.28, 0.146, 0.190, 0.0, 55.4}};
// Block sweep.  A step takes the longer of one wavefront's own rows (c1 each,
// plus lat) and the row updates of the fullest SIMD (c each).
struct BlockFit {
  double t0, lat, c, c1, t1;
};
constexpr BlockFit kBlockFit[4] = {{0.95, 0.0, 0.233, 0.225, 1.84},
                                   {3.47, 0.056, 0.185, 0.248, 0.0},
                                   {4.18, 0.013, 0.225, 0.298, 0.0},
                                   {4.18, 0.013, 0.235, 0.305, 0.0}};

inline double tile_us(int st, const TileShape& t, int L, int cus) {
  const TileFit& f = kTileFit[st];
  const int nodes = t.rx * t.ry, W = (nodes + 63) / 64;
  const int lds = L > 1 ? 16 * W * 64 * kBytes[st] : 0;
  int fit = 28 / W;  // 70 VGPRs: seven wavefronts per SIMD
  if (lds) fit = std::min(fit, 160 * 1024 / lds);
  fit = std::max(1, std::min(fit, 16));
  const int64_t tiles = (int64_t)t.tx * t.ty;
  const int conc = (int)std::min<int64_t>(fit, div_up(tiles, cus));
  const int rounds = div_up(tiles, (int64_t)cus * conc);
  double us = f.t1 + conc * W * (64.0 / t.rx + 1) / f.seg;
  if (t.hx == 0 && t.hy == 0 && L > 1) {  // every step alike (L may be large)
    us += L * (f.lat + f.c * ((W * conc + 3) / 4));
  } else {
    for (int s = 0; s < L; ++s) {
      const int rows = t.ty > 1 ? t.ry - 2 * s : t.ry;
      const int a = std::max(1, std::min(W, (rows * t.rx + 63) / 64));
      us += f.lat + f.c * ((a * conc + 3) / 4);
    }
  }
  return f.t0 + rounds * us;
}

inline double block_us(int st, const BlockShape& b, int L, int cus) {
  BlockFit f = kBlockFit[st];
  // BF16S takes its figures from F16S; its six rows measured slower against its
  // four than modelled.  Of 24 lattices from 62 x 2909 to 1800 x 900 whose plan the
  // factor changes, it gains 2 % on one lattice alone and 8 % on three in flight in the
  // mean (62 x 2909 2.73 -> 2.51 and 1.93 -> 1.59, 1200 x 300 3.32 -> 2.84 and 2.10 ->
  // 1.71; the other way 1024 x 1100 6.1 -> 6.8 and 4.5 -> 5.1, 777 x 600 3.4 -> 3.6).
  if (st == LB_BF16S && b.rows == 6) f.c *= 1.05, f.c1 *= 1.05;
  const int64_t tiles = (int64_t)b.tx * b.ty;
  const int fit = block_fit(st, b.rows, b.waves);
  const int conc = (int)std::min<int64_t>(fit, div_up(tiles, cus));
  const int rounds = div_up(tiles, (int64_t)cus * conc);
  double us = f.t1;
  for (int s = 0; s < L; ++s) {
    const int rows = b.waves * b.rows - 2 * s;
    us += std::max(f.lat + f.c1 * std::min(b.rows, rows), 0.5 * f.lat + f.c * rows * conc / 4.0);
  }
  return f.t0 + rounds * us;
}

// Best tile shape for exactly L steps; us < 0 if there is none.
inline StepPlan best_tile(int st, int nx, int ny, int L, int cus) {
  constexpr int kX[] = {0, 4, 8, 16, 24, 32, 40, 48, 56, 64, 96, 128, 192, 256};
  constexpr int kY[] = {0, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32, 48, 64};
  StepPlan best;
  best.us = -1;
  if (std::max(nx, ny) > kTileMostSide) return best;
  for (int wy : kY) {
    if (wy >= ny) continue;
    TileShape t;
    t.oy = wy == 0 ? ny : div_up(ny, div_up(ny, wy));
    t.ty = div_up(ny, t.oy);
    t.hy = t.ty == 1 ? 0 : L - 1;
    if (t.oy > kTileNodes || t.hy > ny) continue;
    t.ry = t.oy + 2 * t.hy;
    for (int wx : kX) {
      if (wx >= nx) continue;
      t.ox = wx == 0 ? nx : wx;
      t.tx = div_up(nx, t.ox);
      t.hx = t.tx == 1 ? 0 : L - 1;
      if (t.ox > kTileNodes || t.hx > nx) continue;
      t.rx = t.ox + 2 * t.hx;
      if (t.rx * t.ry > kTileNodes) continue;
      if ((int64_t)t.tx * t.ty > 16 * cus) continue;
      const double us = tile_us(st, t, L, cus);
      if (best.us < 0 || us < best.us) {
        best.kind = StepKind::tile;
        best.levels = L;
        best.us = us;
        best.tile = t;
      }
    }
  }
  return best;
}

inline BlockShape block_shape(int nx, int ny, int L, int waves, int rows) {
  BlockShape b;
  b.waves = waves;
  b.rows = rows;
  const int mx = 64 - 2 * (L - 1), my = waves * rows - 2 * (L - 1);
  b.ox = div_up(nx, div_up(nx, mx));
  b.tx = div_up(nx, b.ox);
  b.oy = div_up(ny, div_up(ny, my));
  b.ty = div_up(ny, b.oy);
  return b;
}

// Lattices of many rounds of tiles run at the issue rate of the row updates,
// so the halo share decides: 64 x 64 regions in F32S (54 x 54 stored at six
// steps: 65.6 us per step on 4096^2 against 67.6 at five and 66.9 at seven).
// The 16-bit formats carry the conversions between steps and fill from less
// memory: four steps in 64 x 32 regions (2048^2 F16S: 17.6 us per step, best
// of all shapes; BF16S 4096^2, 64 x 48: 69.4 against 72.9 at six steps).
inline StepPlan block_large(int st, int nx, int ny, int L, int cus) {
  StepPlan p;
  p.kind = StepKind::block;
  p.levels = L;
  const int rows = st == LB_F16S ? block_rows_small(st) : block_rows_big(st);
  p.block = block_shape(nx, ny, L, kBlockWaves, rows);
  p.us = one_launch(p.block.tx, p.block.ty, 64 * kBlockWaves) ? block_us(st, p.block, L, cus) : -1;
  return p;
}
constexpr int block_large_levels(int st) { return st == LB_F16S || st == LB_BF16S ? 4 : 6; }

inline StepPlan best_block(int st, int nx, int ny, int L, int cus) {
  StepPlan best;
  best.us = -1;
  for (int rows : {block_rows_small(st), block_rows_big(st)}) {
    for (int waves = 1; waves <= kBlockWaves; ++waves) {
      if (64 - 2 * (L - 1) < 16 || waves * rows - 2 * (L - 1) < 4) continue;
      const BlockShape b = block_shape(nx, ny, L, waves, rows);
      const int fit = block_fit(st, rows, waves);
      const int64_t tiles = (int64_t)b.tx * b.ty;
      // More than one round only with every SIMD equally loaded.
      if (tiles > (int64_t)cus * fit && waves % 4 != 0) continue;
      if (tiles > (int64_t)3 * cus * fit) continue;
      const double us = block_us(st, b, L, cus);
      if (best.us < 0 || us < best.us) {
        best.kind = StepKind::block;
        best.levels = L;
        best.us = us;
        best.block = b;
      }
    }
  }
  return best;
}

// Flat lattices of many rounds of workgroups (one side short): tiles that cover
// the short side, which then wraps inside LDS, or blocks.  Fitted to 4,700 timed
// launches on 288 lattices of 5e5, 2e6 and 8e6 nodes with a short side of 1 to
// 64, all storages, either orientation; the chosen shape ran at the time of the
// fastest one in the median and within 14 % of it on nine lattices out of ten.
// Per round of the chip a tile or block takes `wave` for every wavefront
// (tiles) or row of a wavefront (blocks) and step, `line` for every 128-byte
// line that it reads or writes, and the latencies of its steps and of itself,
// shared with the workgroups that are resident beside it.
struct FlatFit {
  double t0, wave, line, step, item;
};
constexpr FlatFit kFlatTile[4] = {{5.24, 0.0238, 0.00168, 0.601, 0.748},
                                  {5.94, 0.0306, 0.00119, 0.148, 0.658},
                                  {6.19, 0.0350, 0.00046, 0.130, 0.817},
                                  {6.41, 0.0401, 0.00042, 0.148, 0.631}};
constexpr FlatFit kFlatBlock[4] = {{6.73, 0.0486, 0.00188, 0.508, 0.0},
                                   {2.20, 0.0383, 0.00121, 0.0, 0.0},
                                   {6.71, 0.0444, 0.00063, 0.0, 0.0},
                                   {7.44, 0.0487, 0.00060, 0.061, 0.0}};
inline double flat_us(const FlatFit& f, double waves, double lines, int L, int conc, int64_t tiles,
                      int cus) {
  // In few rounds a last one of some workgroups counts for half of a whole one.
  double r = (double)tiles / ((double)cus * conc);
  if (r < 4) r = 0.5 * (r + std::ceil(r));
  return f.t0 + r * (conc * (f.wave * waves + f.line * lines) + f.step * L + f.item);
}

// Lines of `rows` rows of `columns` values of each of the nine planes; a region
// as wide as the lattice is contiguous.
inline double flat_lines(int st, int columns, int rows, bool whole) {
  const double l = columns * kBytes[st] / 128.0;
  return 9.0 * (whole ? rows * l + 1 : rows * (l + 1));
}

inline StepPlan best_flat(int st, int nx, int ny, int L, int cus) {
  StepPlan best;
  best.us = -1;
  best.levels = L;
  const int h = L - 1;
  const bool wide = nx >= ny;
  const int side = std::min(nx, ny), length = std::max(nx, ny);
  // Four, eight or sixteen wavefronts: the same number on every SIMD.
  for (int W : {4, 8, 16}) {
    const int most = 64 * W / side - 2 * h;
    if (most < 1 || most >= length || h > length || length > kTileMostSide) continue;
    TileShape t{};
    const int out = div_up(length, div_up(length, most));
    t.ox = wide ? out : nx, t.oy = wide ? ny : out;
    t.tx = div_up(nx, t.ox), t.ty = div_up(ny, t.oy);
    t.hx = wide ? h : 0, t.hy = wide ? 0 : h;
    t.rx = t.ox + 2 * t.hx, t.ry = t.oy + 2 * t.hy;
    const int threads = (t.rx * t.ry + 63) / 64 * 64;
    if (!one_launch(t.tx, t.ty, threads)) continue;
    double waves = 0;  // a tall tile's rows run out step by step
    for (int s = 0; s < L; ++s) waves += wide ? threads / 64 : std::max(1, (t.rx * (t.ry - 2 * s) + 63) / 64);
    const int conc = std::max(1, std::min(7 / div_up(threads, 256), 160 * 1024 / (16 * threads * kBytes[st])));
    const double lines = flat_lines(st, t.rx, t.ry, !wide) + flat_lines(st, t.ox, t.oy, !wide);
    const double us = flat_us(kFlatTile[st], waves, lines, L, conc, (int64_t)t.tx * t.ty, cus);
    if (best.us < 0 || us < best.us) best.kind = StepKind::tile, best.us = us, best.tile = t;
  }
  for (int rows : {block_rows_small(st), block_rows_big(st)})
    for (int waves : {4, 5, 6, 8}) {
      if (rows != block_rows_small(st) && waves % 4 != 0) continue;  // uneven SIMDs
      // The 16-bit formats' conversions between steps (48 x 41667 F16S: 12.1 us per
      // step with seven, 10.1 with five; modelled alike).
      if (st >= LB_F16S && L > 5 && best.us >= 0) continue;
      if (64 - 2 * h < 8 || waves * rows - 2 * h < 1) continue;
      const BlockShape b = block_shape(nx, ny, L, waves, rows);
      if (!one_launch(b.tx, b.ty, 64 * waves)) continue;
      double work = 0;
      for (int s = 0; s < L; ++s) work += waves * rows - 2 * s;
      const int conc = block_fit(st, rows, waves);
      const double lines = flat_lines(st, 64, waves * rows, false) + flat_lines(st, b.ox, b.oy, false);
      const double us = flat_us(kFlatBlock[st], work, lines, L, conc, (int64_t)b.tx * b.ty, cus);
      if (best.us < 0 || us < best.us) best.kind = StepKind::block, best.us = us, best.block = b;
    }
  return best;
}

}  // namespace plan_detail

// Lattices that best_flat plans.  Below a million nodes best_tile and best_block
// do better (F32S, us per step: 64 x 7032 4.1 against 5.7, 48 x 16667 4.6 against
// 6.1), but for columns of a few nodes, which best_tile cuts too short (F64 1 x
// 450001 133 against 3).  Blocks of F16S are a good fit from 64 rows on (15001 x
// 100 8.0 against 9.5), the other formats' larger ones are not (BF16S 10.1 against
// 8.7).
inline bool plan_flat(int st, int nx, int ny) {
  const int64_t nodes = (int64_t)nx * ny;
  if (nodes < 1000000) return nx <= 8 && nodes >= 250000;
  return std::min(nx, ny) <= (st == LB_F16S ? 64 : 128);
}

// Wavefronts per strip of the strip pipeline (fused_impl.hpp: 1 or 4) if it
// advances this lattice, 0 if it does not.  A strip
// pays for its halo rows once per strip, a block once per block, so strips
// have the smaller halo share where a lattice fills the chip with long ones;
// below that their pipeline fill (2 K row steps per launch) and the uneven last
// wave cost more.  Measured, us per step, block : strip, one lattice at a time
// (and with three lattices on three streams):
//   F64   512^2 2.84 : 3.48 (2.46 : 2.78), 600^2 4.38 : 4.21 (3.70 : 3.07);
//   F32S  1500^2 12.7 : 13.5 (9.5 : 9.7), 2048^2 18.9 : 19.8 (16.7 : 15.9),
//         2236^2 22.8 : 21.8 (19.8 : 18.7), 2500^2 28.1 : 26.8 (24.7 : 22.9);
//   F16S  1500^2 10.5 : 13.1 (8.7 : 8.9), 2048^2 18.6 : 20.5 (16.6 : 14.7),
//         2236^2 21.7 : 22.7 (19.4 : 17.6), 4096^2 64.9 : 56.5 (63.4 : 48.5);
//   BF16S 2048^2 19.0 : 22.6 (16.9 : 15.9), 2236^2 22.3 : 24.3 (19.8 : 18.8).
// F64 changes over early: its blocks leave two wavefronts per SIMD, which
// cannot hide their loads.  On flat lattices the strips' halo rows (2 K of them
// above and below) or unused columns decide; us per step, tile or block : strips,
// 2e6 and 8e6 nodes:
//   F64 (five numbers)  8 rows 13.1 : 15.7, 50 : 70; 12 rows 15.8 : 15.4, 57 : 57;
//         16 rows 17.9 : 15.0, 63 : 53; 24 rows 16.3 : 12.9, 60 : 44; 24 columns
//         17.0 : 19.5, 63 : 68; 32 columns 18.0 : 15.6, 67 : 52;
//   F32S, 8e6  12 rows 31.5 : 32.9; 20 rows 35.9 : 32.6; 36 rows 38.1 : 33.3;
//   F16S, 8e6  16 rows 32.4 : 33.4; 20 rows 33.1 : 30.8; BF16S 33.2 : 35.5, and
//         24 rows 35.6 : 34.3.
// In FP64 smaller lattices change over at more rows, since tiles and blocks then
// run in few rounds, and strips that store populations (walls, BGK) at others
// than strips of five numbers (BGK 23685 x 19 4.8 : 4.0, walls 107143 x 14 12.4 :
// 14.5).
// The strips of four wavefronts store 244 columns; where a row fills the last one
// badly, the 16-bit formats take strips of one wavefront (52 columns), and F32S,
// which has none, blocks.  us per step, four : one wavefronts (and with three
// lattices on three streams), by the share of columns that hold nodes: F16S 48 x
// 250001 (0.20) 179 : 48; 300 x 20001 (0.61) 32.9 : 24.5; 600 x 10001 (0.82) 26.6
// : 24.1 (21.5 : 22.4); 1500 x 12001 (0.88) 64.5 : 62.0 (57.5 : 60.4); 4096^2
// (0.99) 54.9 : 59.0 (48.9 : 56.5); BF16S 1500 x 12001 75.4 : 65.3 (61.8 : 62.9);
// 2048 x 4096 (0.93) 36.9 : 32.5 (28.6 : 29.9); 4096^2 64.0 : 61.2 (52.8 : 58.5);
// few rows: 250001 x 24 28.8 : 25.2 (21.0 : 23.2), x 48 52.1 : 45.9 (43.1 : 44.0),
// 93751 x 64 29.1 : 26.7 (23.3 : 22.8).
// F32S 48 x 166667, strips of four against blocks: 109 : 36.
inline int plan_strips(int st, int nx, int ny, int coll = LB_COLL_OREG,
                        int bc = LB_BC_PERIODIC) {
  const int64_t nodes = (int64_t)nx * ny;
  if (st != LB_F64) {
    if (nodes < 4500000 || nx <= 36 || ny < 20) return 0;
    const double fill = nx / (244.0 * ((nx + 243) / 244));
    if (st == LB_F32S) return fill < 0.8 ? 0 : 4;
    if (st == LB_F16S) return fill < 0.85 ? 1 : 4;
    return fill < 0.9 || (ny >= 28 && ny < 100) ? 1 : 4;
  }
  if (nodes < 300000 || nx < (nodes >= 4000000 ? 28 : nodes >= 1000000 ? 32 : nodes >= 800000 ? 36 : 37))
    return 0;
  if (coll == LB_COLL_BGK) return ny >= (nodes >= 1000000 ? 12 : 16);
  if (bc == LB_BC_BOUNCEBACK) return ny >= (nodes >= 4000000 ? 16 : 20);
  return ny >= (nodes >= 1000000 ? 12 : nodes >= 800000 ? 14 : 20);
}

// Whether the block sweep runs this lattice in many rounds of workgroups.
inline bool plan_many(int st, int nx, int ny, int cus) {
  using namespace plan_detail;
  const int Lb = block_large_levels(st);
  const StepPlan p = block_large(st, nx, ny, Lb, cus);
  const int fit = block_fit(st, p.block.rows, kBlockWaves);
  return 2 * (int64_t)p.block.tx * p.block.ty > (int64_t)3 * cus * fit;
}

// The plan for one launch of exactly L steps on a lattice that plan_strips
// leaves to the tile and block sweeps; us < 0 if neither takes L steps.
inline StepPlan plan_levels(int st, int nx, int ny, int L, int cus) {
  using namespace plan_detail;
  const int64_t nodes = (int64_t)nx * ny;
  if (plan_flat(st, nx, ny)) return best_flat(st, nx, ny, L, cus);
  StepPlan best;
  best.us = -1;
  // Tiles fill the chip with one small workgroup per CU: up to about 290^2
  // nodes (256^2 F32S: tile 1.3, block 1.6 us per step; 362^2: 2.3 against
  // 1.7).  On flat lattices, which leave most of a block's 64 columns or of
  // its rows empty, at any length.
  if (nodes <= 81920 || std::min(nx, ny) <= 36) best = best_tile(st, nx, ny, L, cus);
  if (L <= 16 && nodes >= 4096) {
    StepPlan b;
    if (plan_many(st, nx, ny, cus)) {
      b.us = -1;
      if (L <= block_large_levels(st)) b = block_large(st, nx, ny, L, cus);
    } else {
      b = best_block(st, nx, ny, L, cus);
    }
    if (b.us >= 0 && (best.us < 0 || b.us < best.us)) best = b;
  }
  return best;
}

// The launch with the least modelled time per step.
inline StepPlan plan_best(int st, int nx, int ny, int cus) {
  StepPlan best;
  best.us = -1;
  const bool flat = plan_flat(st, nx, ny), many = !flat && plan_many(st, nx, ny, cus);
  for (int L : {2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 32, 48, kPlanLevels}) {
    // In many rounds the number of steps is measured, not modelled.
    if (many && std::min(nx, ny) > 36 && L != plan_detail::block_large_levels(st)) continue;
    // Fewer steps than this do not hide what a launch loads (20 x 400000 F32S: 49
    // us per step with three, 36 with five; modelled alike).
    if (flat && L < (st <= LB_F32S ? 4 : 3)) continue;
    const StepPlan p = plan_levels(st, nx, ny, L, cus);
    if (p.us >= 0 && (best.us < 0 || p.us * best.levels < best.us * L)) best = p;
  }
  return best;
}

// Whether a call of n steps leaves the state in the other buffer.  A captured
// call is replayed on the buffers it was captured with, so programs replay calls
// that return to their buffer, and which calls do must not depend on the plan:
// as many launches as strips of K steps would take from 48^2 nodes up (`fused`;
// a remainder in one launch where `remainder` says so, else in single steps),
// one per step below, to the parity.
inline bool swaps_buffers(int64_t n, bool fused, int K, bool remainder) {
  const int64_t rest = n % K;
  return ((!fused ? n : n / K + (remainder ? rest > 0 : rest)) & 1) != 0;
}
constexpr int64_t kFusedFrom = 48 * 48;

// Time of n steps spread evenly over m launches, us(L) being that of one of L
// steps; < 0 if there is no launch of that many (us(L) < 0).
template <class Us>
inline double spread_us(int64_t n, int64_t m, Us&& us) {
  const int64_t q = n / m, longer = n % m;
  const double a = longer > 0 ? us((int)(q + 1)) : 0.0, b = us((int)q);
  return a < 0 || b < 0 ? -1 : a * longer + b * (m - longer);
}

// Launches for n steps: m, or where they would end in the wrong buffer the
// cheaper of one launch fewer (by the factor `gain`) and one more.
template <class Us>
inline int64_t launches_for(int64_t n, int64_t m, bool swap, Us&& us, double gain = 1) {
  if (((m & 1) != 0) == swap) return m;
  if (m >= n) return m - 1;
  if (m <= 1) return m + 1;
  const double fewer = spread_us(n, m - 1, us), more = spread_us(n, m + 1, us);
  return fewer >= 0 && (more < 0 || fewer <= gain * more) ? m - 1 : m + 1;
}

// Launches of at most K steps for n steps of a lattice stored as numbers: the
// cheapest count that ends in the right buffer.  A launch of 1 .. 7 steps takes,
// in units of one of four (us of that one: 560^2 13.4, 1024^2 27, 1700^2 61,
// 2048^2 93, 4096^2 336), 0.6, 0.7, 0.8, 1, 1.26, 1.53 and 1.82 while both buffers
// fit the 256 MB cache, where the steps' arithmetic shows from the first on (1.3, 1.7
// and 2 for the longest on lattices of a few strips per CU, whose halo rows then
// weigh more), and 0.9, 0.9, 0.95, 1, 1.2, 1.43 and 1.66 beyond, where
// memory traffic hides up to four steps.  24 steps in six launches of four, not four of
// six: 1000^2 6.5 against 6.8 us per step, 900 x 700 5.1 against 5.6 (1448^2 and
// 1700^2 2 % more).
inline int64_t number_launches(int64_t n, int K, int64_t nodes, bool swap) {
  static constexpr double kSmall[8] = {0, 0.58, 0.67, 0.8, 1, 1.3, 1.7, 2.0};
  static constexpr double kCached[8] = {0, 0.58, 0.66, 0.79, 1, 1.26, 1.53, 1.82};
  static constexpr double kStreamed[8] = {0, 0.9, 0.9, 0.94, 1, 1.19, 1.43, 1.66};
  const double* const cost = nodes < 600000 ? kSmall : 80 * nodes < 256000000 ? kCached : kStreamed;
  const int64_t least = (n + K - 1) / K;
  int64_t best = n;
  double best_cost = -1;
  for (int l = K; l >= 1; --l)  // counts around those of launches of l steps each
    for (int64_t m = std::max(least, n / l - 1); m <= std::min(n, n / l + 2); ++m) {
      if (((m & 1) != 0) != swap) continue;
      const double c = spread_us(n, m, [&](int L) { return cost[L]; });
      if (best_cost < 0 || c < best_cost || (c == best_cost && m < best)) best_cost = c, best = m;
    }
  return best;
}

// Server launches (serve.hip) advance every resident lattice up to K steps, so
// one work split has to suit the whole set.
//
// Block tiles: the shape of the least modelled time for the set's tiles, 64 x
// 64 regions when they fill the chip, smaller ones when few lattices are
// resident and the launch would otherwise last as long as one workgroup with
// many rows.  This runs on the host whenever the set changes, so all shapes are
// counted in one pass over it (4096 lattices: 42 us, 196 with a pass per shape;
// strips 32, 146).
struct ServeShape {
  int waves, rows;  // block tiles (waves > 0)
  int strip_rows;   // strips (waves = 0): most output rows per work item
};
struct LatticeSize {
  int nx, ny;
};
template <class Sizes>
inline ServeShape serve_blocks(int st, const Sizes& sizes, int K, int cus) {
  using namespace plan_detail;
  struct Candidate {
    int waves, rows;
    unsigned int step;  // output rows of a tile
    int64_t tiles;
  } shapes[6];
  int count = 0;
  for (int waves : {8, 4, 2})
    for (int rows : {block_rows_big(st), block_rows_small(st)})
      if (waves * rows - 2 * (K - 1) >= 4)
        shapes[count++] = {waves, rows, (unsigned int)(waves * rows - 2 * (K - 1)), 0};
  const unsigned int mx = 64 - 2 * (K - 1);
  for (const LatticeSize n : sizes) {
    const int64_t tx = ((unsigned int)n.nx + mx - 1) / mx;
    for (int i = 0; i < count; ++i)
      shapes[i].tiles += tx * (((unsigned int)n.ny + shapes[i].step - 1) / shapes[i].step);
  }
  ServeShape best{kBlockWaves, block_rows_big(st), 0};
  double best_us = -1;
  for (int i = 0; i < count; ++i) {
    BlockShape all{};
    all.tx = (int)std::min<int64_t>(shapes[i].tiles, 1 << 30);
    all.ty = 1;
    all.waves = shapes[i].waves;
    all.rows = shapes[i].rows;
    const double us = block_us(st, all, K, cus);
    if (best_us < 0 || us < best_us) {
      best_us = us;
      best.waves = all.waves;
      best.rows = all.rows;
    }
  }
  return best;
}

// Column strips of equal row blocks.  Blocks of at most 132 rows when the set
// fills the chip (2 - 3 % more capacity than 66), fewer rows when it does
// not: a launch lasts as long as its longest strips, K (rows + 2 K) row
// collisions, times the strips that share a SIMD (the model of fused_cost).
template <class Sizes>
inline int serve_strip_rows(const Sizes& sizes, int K, int width, int cus) {
  constexpr unsigned int kRows[] = {132, 99, 66, 48, 33, 24, 18, 12, 9, 6, 3};
  constexpr int N = sizeof(kRows) / sizeof(kRows[0]);
  int64_t counts[N] = {};
  for (const LatticeSize n : sizes) {
    const int64_t strips = ((unsigned int)n.nx + (unsigned int)width - 1) / (unsigned int)width;
    for (int i = 0; i < N; ++i) counts[i] += strips * (((unsigned int)n.ny + kRows[i] - 1) / kRows[i]);
  }
  int best = 132;
  double best_cost = -1;
  for (int i = 0; i < N; ++i) {
    const int64_t items = counts[i];
    const int most = (int)kRows[i];
    const double w = (double)((items + 4 * cus - 1) / (4 * cus));
    const double cost = w / (1 + 0.08 * (std::min(w, 2.0) - 1)) * (K * (most + 2 * K) - K * (K + 1) + 2 * K);
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = most;
    }
  }
  return best;
}

// Capacity of the 2000-request mix (32^2 to 1024^2), GLUPS, blocks : strips, by
// resident lattices: F16S 256: 180 : 187, 128: 192 : 199, 64: 186 : 187; BF16S
// 168 : 186, 176 : 193, 173 : 181, and 16: 147 : 62, 4: 68 : 10 (strips of fixed
// 132 rows); F32S 256: 185 : 173, 64: 188 : 149.  So F32S takes blocks, the
// 16-bit formats strips from about 60 average lattices on.  F64 takes strips:
// its blocks leave two wavefronts per SIMD.
template <class Sizes>
inline ServeShape serve_shape(int st, const Sizes& sizes, int K, int width, int cus) {
  int64_t nodes = 0;
  for (const LatticeSize n : sizes) nodes += (int64_t)n.nx * n.ny;
  const bool strips = st == LB_F64 || (st != LB_F32S && nodes >= 8000000);
  if (strips) return ServeShape{0, 0, serve_strip_rows(sizes, K, width, cus)};
  return serve_blocks(st, sizes, K, cus);
}

}  // namespace oreg
