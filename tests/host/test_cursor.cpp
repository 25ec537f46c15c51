// CPU replay of the register-held mixing kernel's load cursor (lloid_cursor.h),
// built with the address and undefined-behaviour sanitizers by
// tests/test_host_cursor.py.
#include "lloid_cursor.h"

#include <cstdio>

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
  // window lengths p / q of whole and fractional samples, tpw = ceil(ceil(p / q) / 32) tiles each
  const int64_t lens[][2] = {{1, 1}, {17, 1}, {32, 1}, {65, 2}, {33, 1}, {64, 1}, {191, 3}, {96, 1}, {100, 1}, {321, 2}, {160, 1}};
  for (const auto &l : lens)
    for (int ring = 3; ring <= 4; ++ring)
      for (int64_t w0 = 0; w0 < 9; w0 += 4)
        for (int first = 0; first < 6; ++first)      // tile of the run's first window that the run starts at
          for (int n = 1; n <= 23; ++n) {
            const int64_t p = l[0], q = l[1], len = (p + q - 1) / q;
            const int tpw = (int)((len + 31) / 32);
            if (first >= tpw) continue;
            const WinCursor w(w0, p, q);
            TileLoads ld{w, first, 0};
            TileSource from = TileSource::kNextWindow;   // the kernel starts from the window's resource
            int64_t start = w.start;                     // start of the window whose rows the resource covers
            // ring - 1 tiles ahead, then one more while each of the n is multiplied
            for (int k = 0; k < ring - 1 + n; ++k) {
              CHECK(ld.issued == k);
              if (k < n) {
                const int64_t g = first + k, win = w0 + g / tpw;
                CHECK(from != TileSource::kNone);
                CHECK(start == win * p / q);
                CHECK(ld.win.start == start && ld.win.next_start() == (win + 1) * p / q);
                CHECK(ld.ti == g % tpw);
              } else {
                CHECK(from == TileSource::kNone);        // no tile at or past n reads the operand
              }
              const TileSource next = ld.next(n, tpw);
              if (next == TileSource::kNextWindow) start = ld.win.start;
              if (next != TileSource::kSameWindow) from = next;
            }
          }
  std::printf(g_fail ? "%d checks failed\n" : "ok\n", g_fail);
  return g_fail != 0;
}
