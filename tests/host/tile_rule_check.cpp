// Host-side check of the rules that choose a launch's tile from the step's row count (TileRule): for every row count up to the row limit the workgroups
// of the chosen tile must fit the grid that the launch is sized for, and the choice must be one of least time.  Then the choice itself where it matters:
// steps of few live rows under a large row limit.  Prints "ok <cases>" or the first violation.  Linked against the library, whose rules it calls.
#include <hip/hip_runtime.h>
#include <cstdio>
#include "../../paper_2605_08862_amd/csrc/common.h"

static long cases = 0;

static bool check(const TileRule& r, int M_max, const char* what) {
  for (int M = 0; M <= M_max; ++M, ++cases) {
    const int c = r.choice(M);
    if (c < 0 || c >= r.n) { std::printf("%s: bad choice %d at M=%d\n", what, c, M); return false; }
    if (r.blocks(c, M) > r.grid) { std::printf("%s: grid %d too small for %d at M=%d of %d\n", what, r.grid, r.blocks(c, M), M, M_max); return false; }
    if ((long)r.tile[c].rows * (r.blocks(c, M) / r.tile[c].blocks) < M) { std::printf("%s: rows not covered at M=%d\n", what, M); return false; }
    for (int i = 0; i < r.n; ++i)
      if (r.cost(i, M) < r.cost(c, M)) { std::printf("%s: tile %d is cheaper than %d at M=%d\n", what, i, c, M); return false; }
  }
  return true;
}

int main() {
  struct { Shape s; const char* name; } shapes[] = {
      {{28, 1536, 12, 2, 128, 8960, 151936, BS_BF16, 1e-6f, 1e6f}, "1.5B"},   {{28, 3584, 28, 4, 128, 18944, 152064, BS_BF16, 1e-6f, 1e6f}, "7B"},
      {{2, 256, 6, 2, 128, 512, 1000, BS_BF16, 1e-6f, 1e6f}, "10 heads"},     {{4, 4096, 32, 8, 128, 11008, 8192, BS_BF16, 1e-6f, 1e6f}, "d 4096"},
      {{1, 16384, 128, 16, 128, 65536, 333, BS_BF16, 1e-6f, 1e6f}, "d 16384"}};
  for (const auto& sh : shapes)
    for (int M_max : {641, 645, 663, 702, 816, 1088, 1513, 2176, 4352}) {
      const TileRule q = qkv_rope_rule(sh.s, M_max);
      if (!q.at) { std::printf("%s: no QKV rule at %d\n", sh.name, M_max); return 1; }
      if (!check(q, M_max, sh.name)) return 1;
    }
  for (const auto& sh : shapes)
    for (int M_max : {33, 160, 161, 252, 320, 321, 432, 504, 576, 639, 641, 663, 702, 816, 1088, 1280, 1513, 2176, 4352}) {
      const TileRule g = gate_up_rule(sh.s, M_max);
      if (M_max > 320 && !g.at && !g.fixed) { std::printf("%s: no gate/up rule at %d\n", sh.name, M_max); return 1; }
      if (g.at && !check(g, M_max, sh.name)) return 1;
      if (g.at && g.waves != 4 && g.waves != 8) return 1;
    }
  for (int M_max : {432, 576})
    if (gate_up_rule(shapes[0].s, M_max).at) { std::printf("1.5B, %d rows: a launch of one round of the CUs waits for the row count\n", M_max); return 1; }
  struct { int shape, M_max, M, waves, rows; } glu[] = {{1, 504, 280, 8, 128}, {1, 576, 346, 8, 128}, {1, 714, 134, 8, 160}, {1, 1224, 240, 8, 256}, {0, 639, 197, 8, 96}, {0, 612, 68, 8, 96}, {0, 2176, 128, 4, 192},
                                                        {0, 952, 56, 4, 64}, {3, 432, 108, 8, 96}, {3, 952, 505, 8, 256}};
  for (const auto& e : glu) {
    const TileRule g = gate_up_rule(shapes[e.shape].s, e.M_max);
    const int rows = g.tile[g.choice(e.M)].rows;
    if (rows != e.rows || g.waves != e.waves) {
      std::printf("gate/up of %d of %d rows, %s: %d rows in %d waves, %d in %d expected\n", e.M, e.M_max, shapes[e.shape].name, rows, g.waves, e.rows, e.waves);
      return 1;
    }
  }
  struct { int shape, M_max, M, rows; } qkv[] = {{0, 2176, 128, 32}, {0, 952, 56, 32}, {0, 663, 367, 32}, {1, 714, 134, 32}, {1, 1088, 166, 32}, {2, 1024, 64, 32},
                                                       {2, 2176, 2176, 96}, {2, 2176, 824, 64}};
  for (const auto& e : qkv) {
    const TileRule q = qkv_rope_rule(shapes[e.shape].s, e.M_max);
    const int rows = q.tile[q.choice(e.M)].rows;
    if (rows != e.rows) { std::printf("QKV of %d of %d rows, %s: %d rows per tile, %d expected\n", e.M, e.M_max, shapes[e.shape].name, rows, e.rows); return 1; }
  }
  std::printf("ok %ld\n", cases);
  return 0;
}
