// CPU test of the loud samples' bits and their summary levels (lloid_loud.h)
// against a scan, built with the address and undefined-behaviour sanitizers by
// tests/test_host_loud.py.
#include "lloid_loud.h"

#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

using namespace lloid;

static int g_fail = 0;
#define CHECK(cond)                                              \
  do {                                                           \
    if (!(cond)) {                                               \
      std::printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #cond); \
      ++g_fail;                                                  \
    }                                                            \
  } while (0)

int main() {
  std::mt19937_64 rng(5);
  for (int64_t T : {1, 63, 64, 65, 4095, 4096, 4097, 64 * 4096, 64 * 4096 + 1, 3000001}) {
    CHECK(loud_summary_words(T) <= T / 4032 + 4);
    for (int loud : {0, 1, 2, 40, 5000}) {
      std::vector<int64_t> at;
      for (int k = 0; k < loud; ++k) at.push_back((int64_t)(rng() % (uint64_t)T));
      if (loud == 2) at[0] = 0, at[1] = T - 1;
      std::sort(at.begin(), at.end());
      std::vector<uint64_t> w((size_t)(loud_words(T) + loud_summary_words(T)), 0);
      for (int64_t n : at) w[(size_t)(n >> 6)] |= uint64_t(1) << (n & 63);
      for (int64_t i = 0; i < loud_words(T); ++i)
        if (w[(size_t)i])
          loud_mark(w.data(), T, i, [](uint64_t *p, uint64_t bit) {
            const uint64_t old = *p;
            *p |= bit;
            return old;
          });
      for (int q = 0; q < 4000; ++q) {
        // ranges of every scale around and beside the loud samples
        const int64_t half = (int64_t)(rng() % (uint64_t)(1 + (int64_t(1) << (rng() % 23))));
        const int64_t c = at.empty() || q % 3 == 0 ? (int64_t)(rng() % (uint64_t)T)
                                                   : at[(size_t)(rng() % at.size())] + (q % 2 ? half + 1 : -half);
        const int64_t a = std::min(std::max<int64_t>(0, c - half), T - 1), e = std::max(a, std::min(T - 1, c + half));
        const auto it = std::lower_bound(at.begin(), at.end(), a);
        CHECK(loud_any(w.data(), T, a, e) == (it != at.end() && *it <= e));
      }
    }
  }
  // a range's words: at most two per level
  int levels = 1;
  for (int64_t n = loud_words(int64_t(1) << 28); n > 1; n = loud_words(n)) ++levels;
  CHECK(levels == 5);
  std::printf(g_fail ? "%d checks failed\n" : "ok\n", g_fail);
  return g_fail != 0;
}
