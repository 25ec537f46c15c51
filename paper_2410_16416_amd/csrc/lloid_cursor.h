// Cursors of the register-held mixing kernel over trigger windows and the
// operand tiles of a run.  Plain integer code without HIP types: the kernel
// runs it in scalar registers, a CPU test replays it.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define LLOID_CURSOR __host__ __device__ __forceinline__
#else
#define LLOID_CURSOR inline
#endif

namespace lloid {

// A wave-uniform 64-bit value in scalar registers (64-bit divisions run on the
// vector unit, whose results the compiler takes for divergent).
LLOID_CURSOR int64_t uniform64(int64_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return ((int64_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
#else
  return v;
#endif
}

// Trigger window starts floor(w p / q), w = w0, w0 + 1, ..: a division for the
// first, additions after it.
struct WinCursor {
  int64_t start, rem, step, step_rem, q;
  LLOID_CURSOR WinCursor(int64_t w, int64_t p, int64_t q_) : q(q_) {
    start = uniform64((w * p) / q);
    rem = w * p - start * q;
    step = uniform64(p / q);
    step_rem = p - step * q;
  }
  LLOID_CURSOR int64_t next_start() const { return start + step + (rem + step_rem >= q ? 1 : 0); }
  LLOID_CURSOR void advance() {
    start = next_start();
    rem += step_rem;
    if (rem >= q) rem -= q;
  }
};

// Where the operand rows of the next tile come from.
enum class TileSource { kSameWindow, kNextWindow, kNone };

// The tile loads of one run of n tiles, `tpw` to a window: window `win`, tile
// `ti` of it, `issued` tiles so far.
struct TileLoads {
  WinCursor win;
  int ti, issued;
  // Called after a tile's loads.  Past the run there is no source: the kernel
  // goes on to issue as many loads per tile, all out of an empty resource.  It
  // stays so however many tiles are issued past the run; the windows after it
  // may lie outside the operand.
  LLOID_CURSOR TileSource next(int n, int tpw) {
    ++ti;
    if (++issued >= n) {
      ti = 0;
      return TileSource::kNone;
    }
    if (ti != tpw) return TileSource::kSameWindow;
    ti = 0;
    win.advance();
    return TileSource::kNextWindow;
  }
};

}  // namespace lloid
