// Halos and unused lanes of the plans of lattices of a million nodes and more: no
// plan computes more than three nodes for each one that it stores, and no strips
// leave more than half of their columns empty.
#include <cstdio>
#include <cstdlib>

#include "plan.hpp"

using namespace oreg;

int main() {
  long long plans = 0;
  double most = 0;
  for (int st = 0; st < 4; ++st)
    for (double nodes : {1.0e6, 1.05e6, 1.6e6, 2.5e6, 4.0e6, 8.0e6, 3.0e7, 4.0e8})
      for (int side = 1; side <= 1000; side += side < 70 ? 1 : 37) {
        const int length = (int)(nodes / side) + 1;
        for (int flip = 0; flip < 2; ++flip) {
          const int nx = flip ? side : length, ny = flip ? length : side;
          // strips: the share of their columns that hold nodes
          if (const int waves = plan_strips(st, nx, ny)) {
            const int w = 64 * waves - (st == 0 ? 14 : 12);
            const double fill = nx / ((double)w * ((nx + w - 1) / w));
            if (fill < 0.5) {
              std::printf("FAIL storage %d, %d x %d: strips %.2f full\n", st, nx, ny, fill);
              return 1;
            }
            continue;
          }
          const StepPlan p = plan_best(st, nx, ny, 256);
          double computed = 0;
          if (p.kind == StepKind::tile) computed = (double)p.tile.tx * p.tile.ty * p.tile.rx * p.tile.ry;
          if (p.kind == StepKind::block) computed = (double)p.block.tx * p.block.ty * 64 * p.block.waves * p.block.rows;
          const double ratio = computed / ((double)nx * ny);
          if (ratio > most) most = ratio;
          if (p.us < 0 || ratio > 3) {
            std::printf("FAIL storage %d, %d x %d: %.2f nodes computed per node stored\n", st, nx, ny, ratio);
            return 1;
          }
          ++plans;
        }
      }
  std::printf("plans %lld, at most %.2f\n", plans, most);
  return 0;
}
