// plan3.hpp -- which D3Q27 boxes are stored as ten numbers per node, and the
// tile shape of their sweep (march3.hip), in plain host code.
#pragma once

#include <algorithm>
#include <cstdint>

#include "oreg.h"

namespace oreg {

// Workgroup of the march: threads, nodes of a plane of a tile with its halo
// (one thread and one LDS column each) and output nodes at most.  Eleven
// wavefronts and 64 x 8 outputs beat six and 32 x 8 on every box measured
// (256^3 F64 590 : 710 us): fewer halo nodes, longer rows.
constexpr int kMarchThreads = 704, kMarchRegion = 660, kMarchOut = 512;

// The box in tiles of tx x ty columns, each marched along z in chunks of zc
// planes by one workgroup.  A plane of a tile has (tx + 2) (ty + 2) nodes, one
// halo node per side, of which tx ty are kept.
struct MarchShape {
  int tx, ty, zc;
  int ntx, nty, nzc;
};

inline bool march_shape_ok(const MarchShape& s, int nx, int ny, int nz) {
  return s.tx >= 1 && s.ty >= 1 && s.zc >= 1 &&
         (int64_t)(s.tx + 2) * (s.ty + 2) <= kMarchRegion && s.tx * s.ty <= kMarchOut &&
         (int64_t)s.ntx * s.tx >= nx && (int64_t)s.nty * s.ty >= ny && (int64_t)s.nzc * s.zc >= nz &&
         (int64_t)s.ntx * s.nty * s.nzc * kMarchThreads < 4294967296LL;
}

// Whether a box is stored as ten numbers per node after its first step.  The
// march costs more latency per launch than the population sweep (two phases
// and a barrier per plane), so small boxes keep their populations.  In FP64 the
// population sweep takes one round up to 2048 segments of rows (segments: 64
// nodes each), eight wavefronts per CU: us per step, populations : ten numbers,
// 40^3 (1600 segments) 8.4 : 8.9, 45^3 (2025) 9.7 : 10.7, 250 x 18 x 18 (1296) 10.0
// : 11.0, 46^3 (2116) 13.6 : 11.6, 17 x 28 x 200 (5600) 17.5 : 11.0, 64^3 23.5 :
// 16.8, 256^3 1322 : 552 (and moments 6.4 : 7.9 to 10.3 : 13.0); F32S 17 x 28 x 200
// 8.7 : 9.5, 64^3 12.5 : 11.8 (and diagnostics then 32 : 38), 100 x 84 x 60 25.5 :
// 17.8, 256^3 648 : 352.  The 16-bit formats would store ten FP32 numbers (40 bytes)
// for 27 populations (54), and the march's arithmetic then costs more than the bytes
// save (256^3 BF16S 376 : 417).
// BGK keeps all 27 numbers of a node.
inline bool march_worthwhile(int coll, int st, int64_t cells, int64_t segments = INT64_MAX) {
  if (coll != LB_COLL_OREG) return false;
  if (st == LB_F64) return cells >= 60000 && (segments > 2048 || cells >= 110000);
  if (st == LB_F32S) return cells >= 300000;
  return false;
}

namespace plan_detail {
// Modelled time of a march (us, up to a constant): rounds of workgroups times
// planes times a plane's time, from its wavefronts and the cache lines of its
// rows; fitted to 9,000 launches on ten boxes.
inline double march_us(int st, const MarchShape& s, int cus) {
  const double wg = (double)s.ntx * s.nty * s.nzc / cus;
  const double rounds = wg <= 1 ? 1 : (wg < 3 ? (double)(int64_t)(wg + 0.9999) : wg + 0.3);
  const int w = ((s.tx + 2) * (s.ty + 2) + 63) / 64, ow = (s.tx * s.ty + 63) / 64;
  const int line = st == LB_F64 ? 16 : 32;
  const double lines = (s.ty + 2) * (double)(s.tx + 2 + line) / line +
                       s.ty * ((double)s.tx / line + (s.tx % line != 0));
  const double plane = st == LB_F64 ? 1.22 + 0.106 * w + 0.015 * lines
                                    : 1.08 + 0.048 * w + 0.032 * ow + 0.0047 * lines;
  return 2.0 + rounds * (s.zc + 2) * plane * (1 + 2.0 / s.tx);
}
}  // namespace plan_detail

inline MarchShape march_shape(int st, int nx, int ny, int nz, int cus) {
  auto up = [](int a, int b) { return (a + b - 1) / b; };
  MarchShape best{};
  double best_us = -1;
  const int kx0 = up(nx, 198);
  for (int kx = kx0; kx < kx0 + 24 && kx <= nx; ++kx) {
    MarchShape s;
    s.tx = up(nx, kx);
    s.ntx = up(nx, s.tx);
    const int most = std::min(kMarchRegion / (s.tx + 2) - 2, kMarchOut / s.tx);
    if (most < 1) continue;
    const int ky0 = up(ny, most);
    for (int ky = ky0; ky < ky0 + 6 && ky <= ny; ++ky) {
      s.ty = up(ny, ky);
      s.nty = up(ny, s.ty);
      for (int m = 1; m <= 4; ++m) {
        // as many chunks as m rounds of workgroups take
        const int64_t fill = (int64_t)cus * m / ((int64_t)s.ntx * s.nty);
        const int want = (int)std::max<int64_t>(1, std::min<int64_t>(fill, nz));
        s.zc = up(nz, want);
        s.nzc = up(nz, s.zc);
        if (!march_shape_ok(s, nx, ny, nz)) continue;
        const double us = plan_detail::march_us(st, s, cus);
        if (best_us < 0 || us < best_us) {
          best_us = us;
          best = s;
        }
      }
    }
  }
  return best;
}

// The shape of the diagnostics, whose partial sums are per workgroup: the same on
// every device (and partition of one), so that their order is.
inline MarchShape sums_shape(int st, int nx, int ny, int nz) {
  return march_shape(st, nx, ny, nz, 256);
}

}  // namespace oreg
