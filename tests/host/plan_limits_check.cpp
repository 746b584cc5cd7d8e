// Plans of the longest lattices that lb_create accepts (one side from 4 x 10^8
// nodes to 2^31 - 1): index arithmetic without overflow (this runs under the
// undefined-behaviour sanitizer), regions that fit the workgroup, tiles that
// cover the lattice, and launches of fewer than 2^32 work-items.
#include <cstdio>
#include <cstdlib>

#include "plan.hpp"

using namespace oreg;

static void fail(const char* what, int st, int nx, int ny, int L) {
  std::printf("FAIL %s: storage %d, %d x %d, %d steps\n", what, st, nx, ny, L);
  std::exit(1);
}

static void check(int st, int nx, int ny, int L, const StepPlan& p) {
  if (p.us < 0) return;
  long long tiles = 0, threads = 0;
  if (p.kind == StepKind::tile) {
    const TileShape& t = p.tile;
    if (t.rx < 1 || t.ry < 1 || (long long)t.rx * t.ry > kTileNodes) fail("region", st, nx, ny, L);
    if ((long long)t.tx * t.ox < nx || (long long)t.ty * t.oy < ny) fail("cover", st, nx, ny, L);
    if (nx > 2147483647 - 2 * kTileNodes || ny > 2147483647 - 2 * kTileNodes) fail("tile past an int", st, nx, ny, L);
    tiles = (long long)t.tx * t.ty;
    threads = (t.rx * t.ry + 63) / 64 * 64;
  } else if (p.kind == StepKind::block) {
    const BlockShape& b = p.block;
    if (b.ox < 1 || b.ox + 2 * (L - 1) > 64 || b.oy < 1 || b.oy + 2 * (L - 1) > b.waves * b.rows)
      fail("region", st, nx, ny, L);
    if ((long long)b.tx * b.ox < nx || (long long)b.ty * b.oy < ny) fail("cover", st, nx, ny, L);
    tiles = (long long)b.tx * b.ty;
    threads = 64 * b.waves;
  }
  if (tiles * threads >= 4294967296LL) fail("launch", st, nx, ny, L);
}

int main() {
  long long plans = 0;
  for (int st = 0; st < 4; ++st)
    for (int ny : {1, 2, 3, 4, 8, 17})
      for (int nx : {400000000, 453000001, 500000000, 1000000007, 2147483391, 2147483647}) {
        if ((long long)nx * ny > (st < 2 ? 4294966784LL : 8589933568LL)) continue;
        for (int flip = 0; flip < 2; ++flip) {
          const int a = flip ? ny : nx, b = flip ? nx : ny;
          (void)plan_strips(st, a, b);
          const StepPlan best = plan_best(st, a, b, 256);
          check(st, a, b, best.levels, best);
          for (int L = 2; L <= 16; ++L) check(st, a, b, L, plan_levels(st, a, b, L, 256));
          ++plans;
        }
      }
  // what the server's block launch is cut into
  for (int waves = 1; waves <= kBlockWaves; ++waves)
    if (launch_items(64 * waves) * 64 * waves >= 4294967296LL ||
        (launch_items(64 * waves) + 1) * 64 * waves < 4294967296LL)
      fail("launch items", waves, 0, 0, 0);
  std::printf("plans %lld\n", plans);
  return 0;
}
