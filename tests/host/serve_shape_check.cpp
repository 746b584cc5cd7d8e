// The work split of a set of served lattices equals the one from a pass per shape.
#include <cstdio>
#include <vector>

#include "plan.hpp"

using namespace oreg;
using namespace oreg::plan_detail;

static ServeShape by_shape(int st, const std::vector<LatticeSize>& sizes, int K, int width, int cus) {
  ServeShape best{kBlockWaves, block_rows_big(st), 0};
  double least = -1;
  long long nodes = 0;
  for (const LatticeSize n : sizes) nodes += (long long)n.nx * n.ny;
  if (st == LB_F64 || (st != LB_F32S && nodes >= 8000000)) {
    best = {0, 0, 132};
    for (int most : {132, 99, 66, 48, 33, 24, 18, 12, 9, 6, 3}) {
      long long items = 0;
      for (const LatticeSize n : sizes) items += (long long)div_up(n.nx, width) * div_up(n.ny, most);
      const double w = (double)((items + 4 * cus - 1) / (4 * cus));
      const double cost =
          w / (1 + 0.08 * (std::min(w, 2.0) - 1)) * (K * (most + 2 * K) - K * (K + 1) + 2 * K);
      if (least < 0 || cost < least) least = cost, best.strip_rows = most;
    }
    return best;
  }
  for (int waves : {8, 4, 2})
    for (int rows : {block_rows_big(st), block_rows_small(st)}) {
      if (waves * rows - 2 * (K - 1) < 4) continue;
      long long tiles = 0;
      for (const LatticeSize n : sizes) {
        const BlockShape b = block_shape(n.nx, n.ny, K, waves, rows);
        tiles += (long long)b.tx * b.ty;
      }
      BlockShape all{};
      all.tx = (int)std::min<long long>(tiles, 1 << 30);
      all.ty = 1;
      all.waves = waves;
      all.rows = rows;
      const double us = block_us(st, all, K, cus);
      if (least < 0 || us < least) least = us, best.waves = waves, best.rows = rows;
    }
  return best;
}

int main() {
  unsigned int seed = 1;
  auto random = [&](int n) { return (int)((seed = seed * 1664525u + 1013904223u) >> 8) % n; };
  int checked = 0;
  for (int count : {1, 2, 5, 17, 64, 300, 1500})
    for (int side : {1, 8, 60, 500, 3000, 400000000})
      for (int st = 0; st < 4; ++st)
        for (int rep = 0; rep < 3; ++rep, ++checked) {
          std::vector<LatticeSize> sizes;
          for (int i = 0; i < count; ++i) {
            const int ny = side > 3000 ? 1 + random(3) : 1 + random(side);
            sizes.push_back({1 + random(side), ny});
            if (rep == 1) std::swap(sizes.back().nx, sizes.back().ny);
          }
          const int K = st == LB_F64 ? 7 : 6, width = st == LB_F64 ? 52 : 244;
          const ServeShape a = serve_shape(st, sizes, K, width, 256),
                           b = by_shape(st, sizes, K, width, 256);
          if (a.waves != b.waves || a.rows != b.rows || a.strip_rows != b.strip_rows) {
            std::printf("storage %d, %d lattices up to %d: %d x %d, %d and %d x %d, %d\n", st, count,
                        side, a.waves, a.rows, a.strip_rows, b.waves, b.rows, b.strip_rows);
            return 1;
          }
        }
  std::printf("checked %d\n", checked);
}
