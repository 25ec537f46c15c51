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

static double rounds(int64_t tiles, int64_t steps, int64_t slots, int64_t p) {
  const int64_t r = (tiles * p + slots - 1) / slots, s = (steps + p - 1) / p;
  return (double)r * ((double)s + kMixOverhead);
}

int main() {
  CHECK(mix_parts(0, 8, 256) == 1);
  CHECK(mix_parts(8, 1, 256) == 1);
  CHECK(mix_parts(8, 8, 0) == 1);
  CHECK(mix_parts(256 * 32, 8, 256) == 1);   // whole rounds: nothing to gain
  CHECK(mix_parts(1, 8, 256) == 8);          // one window: a step each
  CHECK(mix_parts(384, 8, 256) > 1);         // one and a half rounds
  std::mt19937 rng(3);
  for (int i = 0; i < 20000; ++i) {
    const int64_t tiles = 1 + rng() % 3000, steps = 1 + rng() % 200, slots = 1 + rng() % 512;
    const int64_t p = mix_parts(tiles, steps, slots);
    CHECK(p >= 1 && p <= steps && p <= 64);
    CHECK(p == 1 || rounds(tiles, steps, slots, p) < 0.96 * rounds(tiles, steps, slots, 1));
    for (int64_t q = 1; q <= steps && q <= 64; ++q)   // no other split is better by more than the margin
      CHECK(rounds(tiles, steps, slots, p) <= rounds(tiles, steps, slots, q) / 0.96 + 1e-9);
  }
  std::printf(g_fail ? "%d checks failed\n" : "ok\n", g_fail);
  return g_fail != 0;
}
