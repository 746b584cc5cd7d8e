// Registers, not LDS, decide how many workgroups of the block sweep a CU holds (but
// for the last two of 28 single wavefronts).
#include <cstdio>

#include "plan.hpp"

int main() {
  using namespace oreg;
  int n = 0;
  for (int st = 0; st < 4; ++st)
    for (int rows : {block_rows_small(st), block_rows_big(st)})
      for (int waves = 1; waves <= kBlockWaves; ++waves, ++n) {
        const int by_registers = 4 * block_waves_per_simd(st, rows) / waves;
        const int fit = block_fit(st, rows, waves);
        if (fit < (by_registers > 26 ? 26 : by_registers < 1 ? 1 : by_registers) ||
            fit * block_lds(st, waves) > 160 * 1024) {
          std::printf("storage %d, %d rows, %d waves: %d fit\n", st, rows, waves, fit);
          return 1;
        }
      }
  std::printf("checked %d shapes\n", n);
}
