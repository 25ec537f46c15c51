// Host-only planning logic of the filtering path: integer range arithmetic of
// the multi-rate resampling, the interpolation hops of a slice, trigger
// windows, the device-memory admission of serving banks and the window
// readiness of a stream.  No HIP types or calls: the runtime uses these, and
// a CPU test (built with address and undefined-behaviour sanitizers) checks
// them against brute force and their invariants.
#pragma once

#include <stdint.h>

#include <deque>
#include <vector>

namespace lloid {

// Half-band resampler: g[n], |n| <= kHalfQ, zero at even n != 0.
constexpr int kHalfQ = 32;
constexpr int kHalfTaps = 2 * kHalfQ + 1;
// Output samples of one interpolation task (32 channels x kUpCols samples).
constexpr int kUpCols = 128;
constexpr int kMaxLevel = 7;       // lowest slice rate f0 / 128
constexpr int kMaxAutocorrHalf = 512;
constexpr int kMaxHops = 4;        // interpolation hops of a level-7 slice: x2, x4, x4, x4

inline int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }
inline int64_t floor_div(int64_t a, int64_t b) { return a >= 0 ? a / b : -((-a + b - 1) / b); }
inline int64_t ceil_div(int64_t a, int64_t b) { return -floor_div(-a, b); }

struct Range {
  int64_t lo = 0, hi = 0;  // absolute indices [lo, hi)
  int64_t size() const { return hi > lo ? hi - lo : 0; }
};

// interpolation reads w[j] with |n - 2j| <= Q and decimation reads u[2k - m]
// with |m| <= Q: the range a level needs from the one above it
inline Range halo_up(Range r) { return {ceil_div(r.lo - kHalfQ, 2), floor_div(r.hi - 1 + kHalfQ, 2) + 1}; }

inline std::vector<Range> need_ranges(int64_t t0, int64_t t1, int n_levels) {
  std::vector<Range> need(n_levels);
  need[0] = {t0, t1};
  for (int k = 1; k < n_levels; ++k) need[k] = halo_up(need[k - 1]);
  return need;
}

// Trigger windows: window w starts at floor(w p / q).
struct Windows {
  int64_t p = 1, q = 1;
  int64_t start(int64_t w) const { return (w * p) / q; }
  int64_t count(int64_t n) const { return ceil_div(n * q, p); }   // windows intersecting [0, n)
};

// Interpolation hops of a slice at `level` for full-rate outputs [t0, t1):
// hop h maps level lev_in[h] to lev_out[h] by r[h] on range out[h] (aligned
// tiles), reading in[h]; the FIR must produce in[0].
struct UpPlan {
  std::vector<int> r, lev_in, lev_out;
  std::vector<Range> in, out;
};
UpPlan up_plan(int64_t t0, int64_t t1, int level);
// Row pitch (elements) of each channel-major low-rate buffer of a slice for
// outputs spanning t_len samples, an upper bound over output positions:
// [0] the FIR output, [h] the output of hop h - 1.
std::vector<int64_t> low_ld(int64_t t_len, int level);

// Device-memory admission of serving banks: banks enter slots in arrival
// order while their bytes fit the budget (0: no limit); the others wait and
// are admitted, still in arrival order, as removals free budget.  A queued
// bank never lets a later one pass it.
class Admission {
 public:
  explicit Admission(int64_t budget = 0) : budget_(budget) {}
  // Add a bank needing `bytes`; returns its slot id and sets *active.  A bank
  // that alone exceeds a nonzero budget is refused: -1.
  int32_t add(int64_t bytes, bool *active);
  // Remove an active or queued slot; false if there is no such slot.
  bool remove(int32_t slot);
  bool active(int32_t slot) const { return slot >= 0 && slot < (int32_t)slots_.size() && slots_[slot].active; }
  bool present(int32_t slot) const { return slot >= 0 && slot < (int32_t)slots_.size() && slots_[slot].present; }
  int64_t used() const { return used_; }
  int64_t budget() const { return budget_; }
  int32_t n_slots() const { return (int32_t)slots_.size(); }
  int32_t n_active() const;
  int32_t n_queued() const { return (int32_t)queue_.size(); }

 private:
  struct S {
    int64_t bytes = 0;
    bool present = false, active = false;
  };
  void admit_queued();
  int64_t budget_ = 0, used_ = 0;
  std::vector<S> slots_;
  std::deque<int32_t> queue_;
};

// Window readiness of a stream: the largest window end wb in (w_next,
// w_next + max_w] such that every window below wb is computable now, or
// w_next when none is.  A window range [w_next, wb) needs full-rate outputs
// [t0, t1) = [start(w_next), min(start(wb), n_end)) plus `margin` samples on
// each side; a slice at `level` whose filter starts `shift` samples (at its
// rate) before the output reads its level up to the need range's end minus
// that shift, which every detector must have computed (avail[level]).
struct ReadySlice {
  int level = 0;
  int64_t shift = 0;   // start tap / decimation factor
  int64_t margin = 0;  // operand samples beyond each end of the outputs
};
struct ReadyState {
  Windows win;
  int64_t w_next = 0;
  int max_w = 1;
  int64_t n_end = -1;                        // data end once flushed (-1 while streaming)
  std::vector<int64_t> pushed;               // per detector: full-rate samples received
  std::vector<std::vector<int64_t>> avail;   // per detector, per level: computed frontier (exclusive)
  std::vector<ReadySlice> slices;            // every slice of every active bank
};
int64_t ready_until(const ReadyState &st);

// Rounds that `units` units (windows, parts of them or runs of tiles) of
// `row_tiles` row tiles (over all jobs) take on `slots` workgroup slots.  All
// row tiles of a unit go to one of the 8 XCDs, units round-robin, so the XCD
// with the most units decides; fewer than 8 units spread over all of them.
inline int64_t mix_rounds(int64_t units, int64_t row_tiles, int64_t slots) {
  if (units < 8 || slots < 8) return ceil_div(units * row_tiles, slots);
  return ceil_div(ceil_div(units, 8) * row_tiles, slots / 8);
}

// Workgroups that share one window of one row tile in the mixing launch:
// `windows` windows of `steps` column steps each.  With p parts per window the
// launch takes mix_rounds of ceil(steps / p) steps, and a workgroup costs about
// kMixOverhead of a step besides (the first chunk's latency, the peaks'
// reduction).  The p with the smallest such time, and 1 unless that gains more
// than 4 %.  Measured on 256 CUs, one workgroup per window against this rule:
// 72 tiles of 8 steps (an 8 s block of 1024 templates) 98 -> 49 us, 384 tiles
// (48 s) in FP32 1880 -> 1487 us and with the SNR series 331 -> 285 us; 8192
// tiles (1024 s) stay whole.
constexpr double kMixOverhead = 0.75;
int mix_parts(int64_t windows, int64_t row_tiles, int64_t steps, int64_t slots);

// Tiles per workgroup of the register-held mixing launch, whose windows hold
// `total` tiles: the run length with the smallest mix_rounds of a run and
// kMixRegOverhead tiles' time (the mixing rows' load, the first tiles'
// latency), of at most kMixRegRun tiles.  341 templates, 40 s in 0.5 s windows,
// 255 runs of 31 tiles: 33 on one XCD's 32 CUs, 102 us; 240 runs of 32, one
// round: 46 us.
constexpr int64_t kMixRegRun = 256;
constexpr double kMixRegOverhead = 4.0;
int64_t mix_reg_run(int64_t total, int64_t row_tiles, int64_t slots);

// Whether the register-held mixing form takes a concatenated K and windows of
// win_len samples (16-bit operands, no SNR series).  Beyond K = 640 its mixing
// fragments do not fit the registers.  Below K = 128 its arithmetic per tile, the
// same for every K, outlasts the products, and the direct-to-LDS form, which
// pays more per window, is faster on long windows.  Register-held against
// direct-to-LDS, 1024 templates on 2^20 samples, windows of 512, 1024, 2048, 4096
// and 16384 samples: K = 32 0.82, 1.09, 1.36, 1.58, 1.83 of its time; K = 64 0.73,
// 0.92, 1.08, 1.22, 1.37; K = 96 0.63, 0.75, 0.85, 0.95, 1.02; K = 128 0.63, 0.77,
// 0.89, 0.96, 1.01 (BF16 within 0.06 of these).
inline bool mix_reg_fits(int kcat, int64_t win_len) {
  if (kcat > 640) return false;
  return kcat >= 128 || win_len <= (kcat < 96 ? 16 * (int64_t)kcat : 4096);
}

// Whether a FIR job of `taps` takes narrow tiles (a quarter of the columns)
// in a launch whose jobs need `work` = sum over jobs of wide tiles x taps, on
// `n_cu` CUs: where a wide tile, on a CU shared by two, lasts longer than the
// launch would with its work spread evenly, so that the longest tiles and not
// the work decide.  A narrow tile reads its fragments from LDS more often per
// product, so a full chip keeps the wide ones.
inline bool fir_narrow(int64_t taps, int64_t work, int64_t n_cu) { return 2 * taps * n_cu > work; }

// BF16 (8-bit significand) pair of a finite FP32 value, as bit patterns:
// hi = x rounded to nearest (ties to even), lo = (x - hi) rounded likewise,
// so that hi + lo carries 16 significant bits of x (the interpolation
// filters of the BF16 operand path are split this way).
void bf16_split(float x, uint16_t *hi, uint16_t *lo);
float bf16_value(uint16_t bits);

}  // namespace lloid
