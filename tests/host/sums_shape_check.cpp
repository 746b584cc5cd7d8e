// The order of the D3Q27 diagnostics' partial sums: workgroups that follow from the
// box alone, whatever the device's CU count, and a node or more for each.
#include <cstdio>

#include "plan3.hpp"

int main() {
  using namespace oreg;
  struct {
    int st, nx, ny, nz, tx, ty, zc;
  } const pinned[] = {
      {0, 64, 64, 64, 64, 8, 2},
      {0, 256, 256, 256, 64, 8, 128},
      {0, 17, 28, 200, 17, 14, 2},
      {0, 300, 1, 500, 150, 1, 4},
      {1, 256, 256, 256, 64, 8, 128},
      {1, 70, 70, 70, 70, 7, 3},
      {1, 100, 84, 60, 100, 4, 5}};
  for (const auto& p : pinned) {
    const MarchShape s = sums_shape(p.st, p.nx, p.ny, p.nz);
    if (s.tx != p.tx || s.ty != p.ty || s.zc != p.zc || !march_shape_ok(s, p.nx, p.ny, p.nz) ||
        (int64_t)s.ntx * s.nty * s.nzc > (int64_t)p.nx * p.ny * p.nz) {
      std::printf("%d x %d x %d: %d x %d, %d planes\n", p.nx, p.ny, p.nz, s.tx, s.ty, s.zc);
      return 1;
    }
  }
  std::printf("checked %d\n", (int)(sizeof pinned / sizeof pinned[0]));
}
