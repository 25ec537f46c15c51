// CPU test of the mixing launch's split rule (lloid_plan.h), built with the
// address and undefined-behaviour sanitizers by tests/test_host_split.py.
#include "lloid_plan.h"

#include <cstdio>
#include <random>

using namespace lloid;

static int g_fail = 0;
#define CHECK(cond)                                              \
  do {                                                           \
    if (!(cond)) {                                               \
      std::printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #cond); \
      ++g_fail;                                                  \
    }                                                            \
  } while (0)

// Rounds by laying every unit's row tiles out on its XCD (or, fewer than 8
// units, on all slots).
static int64_t laid_out(int64_t units, int64_t row_tiles, int64_t slots) {
  if (units < 8 || slots < 8) return (units * row_tiles + slots - 1) / slots;
  int64_t per[8] = {}, most = 0;
  for (int64_t u = 0; u < units; ++u) per[u % 8] += row_tiles;
  for (int64_t x : per) most = x > most ? x : most;
  return (most + slots / 8 - 1) / (slots / 8);
}

int main() {
  CHECK(mix_parts(0, 1, 8, 256) == 1);
  CHECK(mix_parts(8, 1, 1, 256) == 1);
  CHECK(mix_parts(8, 1, 8, 0) == 1);
  CHECK(mix_parts(1024, 8, 8, 256) == 1);   // whole rounds: nothing to gain
  CHECK(mix_parts(1, 1, 8, 256) == 8);      // one window: a step each
  CHECK(mix_parts(48, 8, 8, 256) > 1);      // one and a half rounds
  CHECK(mix_reg_run(0, 8, 256) == 1);
  CHECK(mix_reg_run(2560, 3, 256) == 32);   // 80 runs: 10 units x 3 row tiles on every XCD's 32 CUs
  CHECK(mix_reg_run(64 * 1024, 8, 256) <= kMixRegRun);
  std::mt19937 rng(3);
  for (int i = 0; i < 3000; ++i) {
    const int64_t windows = 1 + rng() % 300, rows = 1 + rng() % 40, steps = 1 + rng() % 100, slots = 1 + rng() % 512;
    auto time = [&](int64_t p) {
      return (double)laid_out(windows * p, rows, slots) * ((double)((steps + p - 1) / p) + kMixOverhead);
    };
    const int64_t p = mix_parts(windows, rows, steps, slots);
    CHECK(p >= 1 && p <= steps && p <= 64);
    CHECK(p == 1 || time(p) < 0.96 * time(1));
    for (int64_t q = 1; q <= steps && q <= 64; ++q)   // no other split is better by more than the margin
      CHECK(time(p) <= time(q) / 0.96 + 1e-9);
    const int64_t total = 1 + rng() % 3000, run = mix_reg_run(total, rows, slots);
    CHECK(run >= 1 && run <= total && run <= kMixRegRun);
    auto time2 = [&](int64_t r) {
      return (double)laid_out((total + r - 1) / r, rows, slots) * ((double)r + kMixRegOverhead);
    };
    for (int64_t r = 1; r <= total && r <= kMixRegRun; ++r) CHECK(time2(run) <= time2(r) + 1e-9);
  }
  std::printf(g_fail ? "%d checks failed\n" : "ok\n", g_fail);
  return g_fail != 0;
}
