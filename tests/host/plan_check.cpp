// Walks lattice sizes and step counts and checks that every plan of plan.hpp
// and plan3.hpp is one that the kernels can run: the region fits the
// workgroup, halos are deep enough and no deeper than the lattice, and the
// tiles cover the lattice without an empty one.  Prints the number of plans,
// or the first broken one.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "plan.hpp"
#include "plan3.hpp"

using namespace oreg;

static void fail(const char* what, int st, int nx, int ny, int L) {
  std::printf("FAIL %s: storage %d, %d x %d, %d steps\n", what, st, nx, ny, L);
  std::exit(1);
}

static void check(int st, int nx, int ny, int L, const StepPlan& p) {
  if (p.us < 0) return;
  if (p.levels != L) fail("levels", st, nx, ny, L);
  if (p.kind == StepKind::tile) {
    const TileShape& t = p.tile;
    if (t.rx < 1 || t.ry < 1 || (long long)t.rx * t.ry > kTileNodes) fail("region", st, nx, ny, L);
    if (t.tx == 1 ? (t.hx != 0 || t.rx != nx) : (t.hx != L - 1 || t.rx != t.ox + 2 * t.hx)) fail("x halo", st, nx, ny, L);
    if (t.ty == 1 ? (t.hy != 0 || t.ry != ny) : (t.hy != L - 1 || t.ry != t.oy + 2 * t.hy)) fail("y halo", st, nx, ny, L);
    if (t.hx > nx || t.hy > ny) fail("halo deeper than the lattice", st, nx, ny, L);
    if ((long long)t.tx * t.ox < nx || (long long)(t.tx - 1) * t.ox >= nx) fail("x cover", st, nx, ny, L);
    if ((long long)t.ty * t.oy < ny || (long long)(t.ty - 1) * t.oy >= ny) fail("y cover", st, nx, ny, L);
  } else if (p.kind == StepKind::block) {
    const BlockShape& b = p.block;
    if (b.waves < 1 || b.waves > kBlockWaves) fail("waves", st, nx, ny, L);
    if (b.rows != block_rows_small(st) && b.rows != block_rows_big(st)) fail("rows", st, nx, ny, L);
    if (b.ox < 1 || b.ox + 2 * (L - 1) > 64) fail("block x", st, nx, ny, L);
    if (b.oy < 1 || b.oy + 2 * (L - 1) > b.waves * b.rows) fail("block y", st, nx, ny, L);
    if ((long long)b.tx * b.ox < nx || (long long)(b.tx - 1) * b.ox >= nx) fail("block x cover", st, nx, ny, L);
    if ((long long)b.ty * b.oy < ny || (long long)(b.ty - 1) * b.oy >= ny) fail("block y cover", st, nx, ny, L);
    if ((long long)b.tx * b.ty * 64 * b.waves >= 4294967296LL) fail("block launch", st, nx, ny, L);
  } else {
    fail("kind", st, nx, ny, L);
  }
}

int main() {
  const int n[] = {1, 2, 3, 5, 7, 8, 16, 31, 32, 33, 36, 37, 48, 63, 64, 65, 100, 127, 128, 129, 200, 255,
                   286, 287, 300, 512, 523, 777, 800, 1024, 1025, 2048, 4096, 16384, 65536, 1000000};
  long long plans = 0;
  for (int st = 0; st < 4; ++st)
    for (int nx : n)
      for (int ny : n) {
        if ((long long)nx * ny > 4294967040LL || plan_strips(st, nx, ny)) continue;
        const StepPlan best = plan_best(st, nx, ny, 256);
        if (best.us < 0) fail("no plan", st, nx, ny, 0);
        check(st, nx, ny, best.levels, best);
        // what lb_step asks for: any number of steps up to the best plan's
        for (int L = 2; L <= best.levels; ++L) {
          const StepPlan p = plan_levels(st, nx, ny, L, 256);
          if (p.us < 0) fail("no plan below the best one", st, nx, ny, L);
          check(st, nx, ny, L, p);
          ++plans;
        }
        for (int cus : {1, 64, 304}) {
          const StepPlan q = plan_best(st, nx, ny, cus);
          if (q.us >= 0) check(st, nx, ny, q.levels, q);
        }
      }
  const int m[] = {1, 2, 3, 7, 16, 17, 40, 64, 66, 100, 197, 198, 199, 256, 300, 512, 1000, 4096, 70000};
  for (int st = 0; st < 2; ++st)
    for (int nx : m)
      for (int ny : m)
        for (int nz : m) {
          const long long cells = (long long)nx * ny * nz;
          if (cells > 4000000000LL || !march_worthwhile(LB_COLL_OREG, st, cells)) continue;
          const MarchShape s = march_shape(st, nx, ny, nz, 256);
          if (!march_shape_ok(s, nx, ny, nz)) fail("march", st, nx, ny, nz);
          if ((s.ntx - 1) * (long long)s.tx >= nx || (s.nty - 1) * (long long)s.ty >= ny ||
              (s.nzc - 1) * (long long)s.zc >= nz)
            fail("empty march tile", st, nx, ny, nz);
          ++plans;
        }
  // server launches: sets of one to many lattices
  for (int st = 0; st < 4; ++st)
    for (int count : {1, 3, 40, 300})
      for (int nx : {1, 32, 65, 500, 1024})
        for (int ny : {1, 33, 200, 1024}) {
          const std::vector<LatticeSize> set(count, LatticeSize{nx, ny});
          const int K = st == 0 ? 7 : 6;
          const ServeShape s = serve_shape(st, set, K, 64 - 2 * K, 256);
          if (s.waves == 0 ? s.strip_rows < 3
                           : (s.waves > kBlockWaves || s.waves * s.rows - 2 * (K - 1) < 4 || st == 0 ||
                              (s.rows != block_rows_small(st) && s.rows != block_rows_big(st))))
            fail("server split", st, nx, ny, count);
          ++plans;
        }
  std::printf("plans %lld\n", plans);
  return 0;
}
