// Host-side check of the rule that chooses the attention chunk size (attn_chunk_candidate, attn_chunk_cost): the plan
// kernel's choice, replayed with exact chunk counts on equal and ragged batches.
//   * every cost is a time: at least one task's fixed cost, whichever branch it comes from;
//   * the work list holds the chosen chunks, and no sequence has more than 512 of them;
//   * small ragged batches that fit the chip in one round of reasonable pieces are not cut into a second round;
//   * a long ragged batch is cut near the fair share of a workgroup and never far above it.
// Prints "ok <cases>" or the first violation.
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdio>
#include <vector>
#include "../../paper_2605_08862_amd/csrc/common.h"

struct Pick { int cht, tasks, max_chunks; bool fits, cost_ok; };

// quantile of the normal law by bisection of erf
static double z_of(double q) {
  double lo = -8, hi = 8;
  for (int i = 0; i < 80; ++i) { const double m = (lo + hi) / 2; (0.5 * (1 + std::erf(m / std::sqrt(2.0))) < q ? lo : hi) = m; }
  return lo;
}
static std::vector<int> batch(int n, double context, double sigma, int k) {
  std::vector<int> t;
  for (int b = 0; b < n; ++b) t.push_back(((int)std::fmin(context * std::exp(sigma * z_of((b + 0.5) / n)), 32768.0) + k + 1 + kTile - 1) / kTile);
  return t;
}
static Pick pick(const AttnPlan& a, const std::vector<int>& t) {
  int T = 0, mx = 0;
  for (int n : t) { T += n; mx = n > mx ? n : mx; }
  const int B = (int)t.size(), cap = attn_item_capacity(B, a.s_min);
  int floor_cht = (T + (cap - B) - 1) / (cap - B);
  if ((mx + 511) / 512 > floor_cht) floor_cht = (mx + 511) / 512;
  if (floor_cht < 1) floor_cht = 1;
  auto items_of = [&](int cht) { int s = 0; for (int n : t) s += (n + cht - 1) / cht; return s; };
  Pick r{0, 0, 0, true, true};
  float best = INFINITY;
  for (int i = 0; i < kAttnCandidates; ++i) {
    const int cht = attn_chunk_candidate(a, i, T, mx, floor_cht);
    const float c = attn_chunk_cost(a, cht, items_of(cht), T, mx, B);
    if (!(c >= a.c_item)) r.cost_ok = false;
    if (c < best || (c == best && cht > r.cht)) { best = c; r.cht = cht; }
  }
  r.tasks = (int)(items_of(r.cht) * a.pairs);
  r.max_chunks = (mx + r.cht - 1) / r.cht;
  r.fits = items_of(r.cht) <= cap;
  return r;
}
int main() {
  long cases = 0;
  const struct { int Hkv, tiles, qb; } kinds[] = {{4, 4, 1}, {2, 4, 1}, {4, 2, 1}, {4, 1, 2}, {2, 1, 2}, {8, 1, 1}};
  for (const auto& kd : kinds)
    for (int D : {64, 128})
      for (int B : {1, 2, 3, 8, 16, 61, 128, 500, 4096})
        for (double ctx : {1.0, 40.0, 300.0, 4096.0, 20000.0})
          for (double sigma : {0.0, 0.3, 1.0, 2.0}) {
            AttnPlan a{};
            a.s_min = (256 + kd.Hkv * kd.qb - 1) / (kd.Hkv * kd.qb);
            attn_plan_constants(a, kd.tiles, kd.qb, kd.Hkv, D);
            const Pick r = pick(a, batch(B, ctx, sigma, 16));
            ++cases;
            if (!r.cost_ok || !r.fits || r.max_chunks > 512 || r.cht < 1) {
              std::printf("Hkv %d tiles %d D %d B %d ctx %g sigma %g: chunk %d, fits %d, costs %d\n", kd.Hkv, kd.tiles, D, B, ctx, sigma, r.cht, r.fits, r.cost_ok);
              return 1;
            }
          }
  AttnPlan w{};
  w.s_min = 64;
  attn_plan_constants(w, 4, 1, 4, 128);                  // wide kernel, 4 KV heads
  const struct { int B; double ctx, sigma; } small[] = {{16, 128, 1.0}, {8, 300, 1.0}, {3, 700, 1.0}, {3, 8000, 1.0}, {32, 1000, 0.3}, {40, 200, 0.3}};
  for (const auto& s : small) {
    const Pick r = pick(w, batch(s.B, s.ctx, s.sigma, 16));
    ++cases;
    if (r.tasks > kAttnWorkgroups) { std::printf("batch %d x %g: chunk %d gives %d tasks\n", s.B, s.ctx, r.cht, r.tasks); return 1; }
  }
  const std::vector<int> lt = batch(128, 4096, 1.0, 16);
  double T = 0;
  for (int n : lt) T += n;
  const Pick r = pick(w, lt);
  const double fair = T * w.pairs / kAttnWorkgroups;
  ++cases;
  if (r.cht < 0.5 * fair || r.cht > 1.1 * fair) { std::printf("long batch: chunk %d, fair share %.0f\n", r.cht, fair); return 1; }
  std::printf("ok %ld\n", cases);
  return 0;
}
