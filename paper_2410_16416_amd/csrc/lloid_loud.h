// Bits of the loud samples of a conditioned block, with levels of summary bits
// above them: bit i of a level is set when word i of the level below is not
// zero, up to a level of one word.  Whether a range of samples holds a loud one
// then takes at most two words per level (five levels for 2^28 samples),
// whatever the range's length.  Plain integer code without HIP types: kernels
// and a CPU test use it.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define LLOID_LOUD __host__ __device__ __forceinline__
#else
#define LLOID_LOUD inline
#endif

namespace lloid {

LLOID_LOUD int64_t loud_words(int64_t bits) { return (bits + 63) >> 6; }

// Words of the levels above the samples' own, which lie behind those.
LLOID_LOUD int64_t loud_summary_words(int64_t T) {
  int64_t total = 0;
  for (int64_t n = loud_words(T); n > 1;) total += n = loud_words(n);
  return total;
}

// Word `i` of the samples' level (at w, T samples) is not zero: set its summary
// bits.  or_word(p, bit) sets *p |= bit and returns the old word; whoever finds
// one that was not zero leaves the levels above to the one who set it first.
template <typename Or> LLOID_LOUD void loud_mark(uint64_t *w, int64_t T, int64_t i, Or or_word) {
  for (int64_t n = loud_words(T); n > 1; i >>= 6) {
    w += n;
    n = loud_words(n);
    if (or_word(w + (i >> 6), uint64_t(1) << (i & 63))) return;
  }
}

// Is any of the samples a..e (0 <= a <= e < T) loud?
LLOID_LOUD bool loud_any(const uint64_t *w, int64_t T, int64_t a, int64_t e) {
  for (int64_t n = loud_words(T);; n = loud_words(n)) {
    const int64_t wa = a >> 6, we = e >> 6;
    const uint64_t ma = ~uint64_t(0) << (a & 63), me = ~uint64_t(0) >> (63 - (e & 63));
    if (wa == we) return (w[wa] & ma & me) != 0;
    if ((w[wa] & ma) | (w[we] & me)) return true;
    if (we - wa < 2) return false;
    w += n;   // whole words between them: bits of the level above
    a = wa + 1;
    e = we - 1;
  }
}

}  // namespace lloid
