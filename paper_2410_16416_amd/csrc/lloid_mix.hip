// Mixing and window peaks with the mixing rows held in registers (16-bit
// operands, concatenated K up to 640, below 128 only with short windows, no SNR
// series: mix_reg_job).
//
// Y[c, n] = sum_k M[c, k] O[n, k]; rows 2i and 2i + 1 (cos, sin) of template i
// land in the same lane, so |z|^2 and the running per-template peak stay in
// registers.  A workgroup of four waves (one per SIMD, the whole register
// file each) owns 256 mixing rows for a run of 32-sample operand tiles; a
// wave holds the MFMA fragments of its 64 rows for every k-step and streams
// the tiles through LDS, so the only LDS traffic is the operand (0.5 KB read
// per 32x32x16 MFMA against 0.75 for 64 x 128 wave tiles with both operands
// in LDS, and half the writes) and a tile takes one barrier.  Two accumulator
// sets: the |z|^2 and peak arithmetic of one tile runs between the MFMAs of
// the next.
//
// What bounds it: the MFMAs at the clock that their power leaves (K = 480:
// 1.28 PFLOP/s, what the library's 8192^3 FP16 product reaches on the same
// card), and below K of some 150 the 80 vector instructions per tile.
// Measured, 1024 templates x 256 s, against k_mix_dl: K = 480 970 -> 798 us,
// 352 753 -> 620, 256 559 -> 477, 160 422 -> 366, 96 311 -> 282; 1024 s at K =
// 480 3.86 -> 3.04 ms (BF16, 200 s: 827 -> 603 us).  A k-step's comparisons all
// come before its selects (a select waits two slots for its comparison) and a
// window's length is worked out once per window, not per tile: 312 -> 282 us at
// K = 96, 3.11 -> 3.04 ms for the 1024 s.  A deeper ring is slower at a small K (16
// tiles, K = 96: 380 us).  On the way: with the
// arithmetic of a tile left after its MFMAs 3.36 ms, with the mixing fragments
// in the vector registers' spare places and copied for each use 3.66 ms.  The
// SNR series stays with k_mix_dl: stores of 256 bytes per template and tile
// here against 2 KB there, a call of 48 s and 1024 templates 535 against 485 us.
//
// A K up to 512 fills the accumulation registers.  Up to 640 the last k-steps'
// fragments take 64 of the vector registers and the ring has three tiles
// (two forms, of 576 and 640; a longer K would spill).  Ten uneven banks of 64 s, two of
// them with K = 544 and 640: 1335 us and 386 us in k_mix_dl -> 1636 us; a serving
// tick of 12 banks, 81 + 62 us -> 122 us in one launch.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lloid_cursor.h"
#include "lloid_device.h"
#include "lloid_internal.h"

namespace lloid {

namespace {

typedef __attribute__((address_space(3))) void lds_void;

// Combine op over the 32 lanes of each half-wave: in quads, octets and rows of
// 16 by DPP moves, then the two rows.
template <typename F> __device__ __forceinline__ int half_wave_reduce(int v, F op) {
  v = op(v, __builtin_amdgcn_update_dpp(v, v, 0xb1, 0xf, 0xf, false));    // quad_perm [1, 0, 3, 2]
  v = op(v, __builtin_amdgcn_update_dpp(v, v, 0x4e, 0xf, 0xf, false));    // quad_perm [2, 3, 0, 1]
  v = op(v, __builtin_amdgcn_update_dpp(v, v, 0x141, 0xf, 0xf, false));   // row_half_mirror
  v = op(v, __builtin_amdgcn_update_dpp(v, v, 0x140, 0xf, 0xf, false));   // row_mirror
  return op(v, __builtin_amdgcn_ds_swizzle(v, 0x401f));                   // lane ^ 16
}

// Operand tiles in LDS, all but one ahead of the one multiplied.
constexpr int ring_tiles(int nks) { return nks <= 32 ? 4 : 3; }
constexpr int kRegSteps = 32;   // k-steps whose mixing fragments fill the accumulation registers

// A divisor of the k-steps that covers an LDS read's latency (a k-step is 64
// cycles of MFMAs), where there is one.
constexpr int read_ahead(int nks) {
  for (int d = 5; d <= 13; ++d)
    if (nks % d == 0) return d;
  return nks;
}

template <int NKS> struct MixRegShape {
  static constexpr int P = 2 * NKS + 1;                    // 16-byte chunks per LDS row: odd, so 16 rows start on distinct banks
  static constexpr int LPW = (32 * P + 255) / 256;         // load instructions per wave and tile
  static constexpr int TILE = LPW * 4096;
  static constexpr int R = ring_tiles(NKS);
  static constexpr int LDS = R * TILE;
  static constexpr int D = read_ahead(NKS);   // k-steps read ahead
  static_assert(NKS % D == 0, "k-steps in whole turns of the read-ahead");
};

// Units of job jb: window w has jb.tpw tiles (the longest window's; a shorter
// one's last tiles are empty), numbered g = (window in job) tpw + tile; this
// workgroup takes g0 <= g < g1 of row tile rt.
template <typename T, int NKS>
__device__ __forceinline__ void mix_reg_tiles(const MixJob &jb, int rt, int64_t g0, int64_t g1, char *lds) {
  typedef typename Op<T>::vec vec;
  typedef MixRegShape<NKS> S;
  constexpr int P = S::P, LPW = S::LPW, TILE = S::TILE, kRing = S::R;
  const int lane = threadIdx.x & 63, fr = lane & 31, fh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kld = jb.kld, tpw = jb.tpw;
  const int cpr = jb.kcat / 8;   // 16-byte chunks of an operand row (the rest of 2 NKS: zeros)
  const int pitch = kld * 2;
  const int64_t r0 = (int64_t)rt * 256 + 64 * wave;

  // mixing fragments: rows r0 + 32 mt + fr, k = 16 ks + 8 fh .. + 7 (zeros past the last row)
  vec af[2][NKS];
  {
    const __amdgpu_buffer_rsrc_t ra =
        make_rsrc((const T *)jb.mix + r0 * kld, (jb.rows - r0) * (int64_t)pitch);
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      const int vo = (32 * mt + fr) * pitch + fh * 16;
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks)
        af[mt][ks] = __builtin_bit_cast(
            vec, __builtin_amdgcn_raw_buffer_load_b128(ra, vo, ks * 32, 0));
    }
    // they live in the accumulation registers, which the MFMAs read directly;
    // the sums and everything the vector unit touches stay in the others
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int ks = 0; ks < (NKS < kRegSteps ? NKS : kRegSteps); ++ks) asm volatile("" : "+a"(af[mt][ks]));
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int ks = kRegSteps; ks < NKS; ++ks) asm volatile("" : "+v"(af[mt][ks]));
  }

  // operand loads: load i of a wave fills LDS chunks 64 (4 i + wave) + lane of
  // a tile = row c / P, position c % P (the pad position and rows past 31 load
  // zeros)
  int vo[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int c = 64 * (4 * i + wave) + lane;
    const int row = c / P, q = c - row * P;
    vo[i] = (row < 32 && q < cpr) ? row * pitch + q * 16 : 0x7ff00000;
  }
  const int n = (int)(g1 - g0);
  const int64_t wl0 = uniform64(g0 / tpw);
  WinCursor wc(jb.w0 + wl0, jb.win_p, jb.win_q);   // window and tile of the products
  int tc = (int)(g0 - wl0 * tpw);
  TileLoads ld{wc, tc, 0};                         // those of the loads
  auto window_len = [&](const WinCursor &w) __attribute__((always_inline)) {
    return __builtin_amdgcn_readfirstlane((int)(min(w.next_start(), jb.n_end) - w.start));
  };
  auto window_rsrc = [&](const WinCursor &w) __attribute__((always_inline)) {
    const int64_t we = min(w.next_start(), jb.n_end);
    return make_rsrc((const T *)jb.ocat + (w.start - jb.ocat_abs0) * (int64_t)kld, (we - w.start) * (int64_t)pitch);
  };
  __amdgpu_buffer_rsrc_t rb = window_rsrc(ld.win);
  auto issue_one = [&](int i) __attribute__((always_inline)) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void *)(lds + (ld.issued % kRing) * TILE + wave * 1024 + i * 4096),
                                             16, vo[i], ld.ti * 32 * pitch, 0, 0);
  };
  auto issue_next = [&]() __attribute__((always_inline)) {
    const TileSource from = ld.next(n, tpw);
    // past the run: an empty resource, so that every tile adds LPW loads (of zeros)
    if (from == TileSource::kNone) rb = make_rsrc(jb.ocat, 0);
    else if (from == TileSource::kNextWindow) rb = window_rsrc(ld.win);
  };
#pragma unroll
  for (int t = 0; t < kRing - 1; ++t) {
#pragma unroll
    for (int i = 0; i < LPW; ++i) issue_one(i);
    issue_next();
  }

  VN best[2][8];
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int p = 0; p < 8; ++p) best[mt][p] = VN{-1.f, 0x7fffffff};
  };
  clear();
  int64_t w_prev = 0;            // window of the tile whose peaks are taken next
  int rel_prev = 0, len_prev = 0;
  // accumulator pair e = 0..15 of the previous tile: template row pair (mt, p) = (e / 8, e % 8)
  auto pair_v = [&](const f32x16 (&acc)[2], int e) __attribute__((always_inline)) {
    const float re = acc[e >> 3][2 * (e & 7)], im = acc[e >> 3][2 * (e & 7) + 1];
    return __builtin_fmaf(re, re, im * im);
  };
  // (columns past the window's end are zeros, |z|^2 = 0: they replace only a
  // lane's initial -1 and are dropped by their sample in flush())
  auto pair_best = [&](int e, float v, int rel) __attribute__((always_inline)) {
    const int mt = e >> 3, p = e & 7;
    if (v > best[mt][p].v) best[mt][p] = VN{v, rel};
  };
  // (a pair's peak stays here, between the MFMAs: the compiler would move it past them)
  auto pin = [&](int e) __attribute__((always_inline)) {
    asm volatile("" : "+v"(best[e >> 3][e & 7].v), "+v"(best[e >> 3][e & 7].n));
  };
  // window peaks: each half-wave's 32 columns of every pair, larger |z|^2
  // first, then lower sample; lane fr of a half then writes pair fr
  auto flush = [&]() __attribute__((always_inline)) {
    VN mine{-1.f, 0x7fffffff};
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int p = 0; p < 8; ++p) {
        VN q = best[mt][p];
        if (q.n >= len_prev) q = VN{-1.f, 0x7fffffff};
        const float v = __int_as_float(half_wave_reduce(__float_as_int(q.v), [](int x, int y) {
          return __float_as_int(fmaxf(__int_as_float(x), __int_as_float(y)));
        }));
        const int k = half_wave_reduce(q.v == v ? q.n : 0x7fffffff, [](int x, int y) { return min(x, y); });
        if (fr == 8 * mt + p) mine = VN{v, k};
      }
    const int p = fr & 7;
    const int64_t i = (r0 + 32 * (fr >> 3) + 8 * (p >> 1) + 4 * fh + 2 * (p & 1)) >> 1;
    if (fr < 16 && i < jb.n_templates) put_peak(jb, i, w_prev, mine);
    clear();
  };
  bool last = false;   // the previous tile was its window's (or the run's) last
  int64_t w_cur = jb.w0 + wl0;
  int len_cur = window_len(wc), done = 0;
  // one tile: MFMAs into acc, the previous tile's peaks from prev between them.
  // Its first D k-steps' fragments have been read before the last tile's end,
  // and it reads the next one's (which the barrier at its own start has shown
  // to be in), so that no tile starts with an LDS latency.
  constexpr int D = S::D;
  constexpr int EPK = (16 + NKS - 1) / NKS;   // pairs per k-step
  vec b[D];   // k-step ks in b[ks % D]; D divides NKS, so the next tile's first k-steps fit the same places
  auto frag = [&](int t, int ks) __attribute__((always_inline)) {
    return *(const vec *)(lds + (t % kRing) * TILE + (fr * P + fh) * 16 + ks * 32);
  };
  auto sync = [&]() __attribute__((always_inline)) {
    // this wave's part of the next tile is in; then every wave's, and the
    // buffer of the tile before this one is free.  Not __syncthreads, which
    // would wait for every load.
    asm volatile("" ::: "memory");
    constexpr int V = LPW * (kRing - 3);
    __builtin_amdgcn_s_waitcnt(0x0f70 | (V & 15) | ((V >> 4) << 14));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto tile = [&](f32x16 (&acc)[2], const f32x16 (&prev)[2]) __attribute__((always_inline)) {
    sync();
    const int rel = rel_prev + fr;
    // A wave issues one instruction at a time and a 32x32x16 MFMA lasts eight
    // issue slots: a pair's arithmetic is split over the two MFMAs of a
    // k-step, and the loads go out one per k-step.
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      float v[EPK];
      __builtin_amdgcn_sched_barrier(0);
      acc[0] = Op<T>::mfma(af[0][ks], b[ks % D], ks == 0 ? f32x16{} : acc[0]);
#pragma unroll
      for (int q = 0; q < EPK; ++q)
        if (ks * EPK + q < 16) v[q] = pair_v(prev, ks * EPK + q);
      if (ks >= 1 && ks <= LPW) issue_one(ks - 1);
      __builtin_amdgcn_sched_barrier(0);
      acc[1] = Op<T>::mfma(af[1][ks], b[ks % D], ks == 0 ? f32x16{} : acc[1]);
      b[ks % D] = ks + D < NKS ? frag(done, ks + D) : frag(done + 1, ks + D - NKS);
#pragma unroll
      for (int q = 0; q < EPK; ++q)
        if (ks * EPK + q < 16) pair_best(ks * EPK + q, v[q], rel);
#pragma unroll
      for (int q = 0; q < EPK; ++q)
        if (ks * EPK + q < 16) pin(ks * EPK + q);
    }
    static_assert(LPW < NKS, "a load per k-step");
    issue_next();
    __builtin_amdgcn_sched_barrier(0);
    if (last) flush();
    // this tile is the next one's previous
    w_prev = w_cur;
    rel_prev = 32 * tc;
    len_prev = len_cur;
    ++done;
    ++tc;
    last = tc == tpw || done == n;
    if (tc == tpw) {
      tc = 0;
      ++w_cur;
      wc.advance();
      len_cur = window_len(wc);
    }
  };
  // tile 0 is in (the first tile's own barrier then shows tile 1)
  asm volatile("" ::: "memory");
  constexpr int V0 = LPW * (kRing - 2);
  __builtin_amdgcn_s_waitcnt(0x0f70 | (V0 & 15) | ((V0 >> 4) << 14));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int ks = 0; ks < D; ++ks) b[ks] = frag(0, ks);
  f32x16 a0[2], a1[2];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int e = 0; e < 16; ++e) a0[mt][e] = a1[mt][e] = __builtin_nanf("");   // no previous tile: no |z|^2 compares greater
  int i = 0;
  for (; i + 2 <= n; i += 2) {
    tile(a0, a1);
    tile(a1, a0);
  }
  const bool odd = i < n;
  if (odd) tile(a0, a1);
  const int rel = rel_prev + fr;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    if (odd) pair_best(e, pair_v(a0, e), rel);
    else pair_best(e, pair_v(a1, e), rel);
  }
  flush();
  __builtin_amdgcn_s_waitcnt(0x0f70);   // the zeros past the run have landed
}

template <typename T>
__global__ __launch_bounds__(256, 1) void k_mix_reg(const MixJob *__restrict__ jobs, int n_jobs) {
  __shared__ __attribute__((aligned(1024))) char lds[MixRegShape<32>::LDS];
  static_assert(MixRegShape<36>::LDS <= MixRegShape<32>::LDS && MixRegShape<40>::LDS <= MixRegShape<32>::LDS, "the largest ring");
  const MixJob &jb = jobs[find_job(jobs, n_jobs, blockIdx.x)];
  const int64_t b = (int64_t)blockIdx.x - jb.item0;
  // XCD-aware order as in mix_unit: all row tiles of one run on one XCD
  const int64_t total = jb.nw * jb.tpw, units = uniform64((total + jb.run - 1) / jb.run);
  const bool wide = units >= 8;
  const int64_t slot = wide ? b >> 3 : b, q = uniform64(slot / jb.n_rtiles);
  const int rt = (int)(slot - q * jb.n_rtiles);
  const int64_t u = wide ? q * 8 + (b & 7) : q;
  if (u >= units) return;
  const int64_t g0 = u * jb.run, g1 = min(total, g0 + jb.run);
  // the concatenated K is a multiple of 32: one compiled form per k-step count
  switch (jb.kcat / 32) {
#define MIX_REG(N) case N: mix_reg_tiles<T, 2 * N>(jb, rt, g0, g1, lds); break;
    MIX_REG(1) MIX_REG(2) MIX_REG(3) MIX_REG(4) MIX_REG(5) MIX_REG(6) MIX_REG(7) MIX_REG(8)
    MIX_REG(9) MIX_REG(10) MIX_REG(11) MIX_REG(12) MIX_REG(13) MIX_REG(14) MIX_REG(15) MIX_REG(16)
#undef MIX_REG
    case 17: case 18: mix_reg_tiles<T, 36>(jb, rt, g0, g1, lds); break;
    case 19: case 20: mix_reg_tiles<T, 40>(jb, rt, g0, g1, lds); break;
  }
}

}  // namespace

hipError_t launch_mix_reg(lloid_dtype t, const MixJob *jobs, int n_jobs, int64_t n_items, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  auto go = [&](auto z) {
    k_mix_reg<decltype(z)><<<(unsigned)n_items, 256, 0, s>>>(jobs, n_jobs);
    return hipGetLastError();
  };
  switch (t) {
    case LLOID_F16: return go(_Float16{});
    case LLOID_BF16: return go(__bf16{});
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lloid
