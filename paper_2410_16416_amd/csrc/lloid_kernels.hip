// gfx950 kernels of the LLOID filtering path.
//
// Stages (the method's order, Sec. II.A): strain conversion, half-band
// decimation to every slice rate, the per-slice FIR bank as a sliding-window
// GEMM on MFMA, interpolation of the low-rate orthogonal SNR to the full
// rate, the mixing GEMM over the concatenated basis with a fused complex-SNR
// and per-window peak epilogue, and trigger compaction (Sec. II.B: only the
// triggers leave the device).  FP64 arithmetic appears only in the sigma^2 sums
// (FP64 inputs are converted once).
#include <hip/hip_runtime.h>
#include <type_traits>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <climits>
#include <cstdlib>

#include "lloid_device.h"
#include "lloid_internal.h"
#include "lloid_loud.h"

namespace lloid {

// ---------------------------------------------------------- small kernels

// First kernel of a call: the descriptor tables from (device-visible) host
// memory into device memory, cleared counters, and the strain in FP32 with
// zeros outside [0, n) and a flag on samples that are not finite.  One launch
// for what were a copy, a fill and a conversion: on small blocks each cost
// its launch (4 to 9 us), not its bytes.  Workgroups [0, tab_blocks) copy 16
// bytes per thread, the next zero_blocks clear, the rest convert.  The flag
// may lie in host memory: a plain store of the same value by whoever finds one.
template <typename TI>
__global__ __launch_bounds__(256) void k_ingest(IngestArgs a, int tab_blocks, int zero_blocks) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if ((int)blockIdx.x < tab_blocks) {
    if (t < a.tab_vecs) ((uint4 *)a.tab_dst)[t] = ((const uint4 *)a.tab_src)[t];
    return;
  }
  if ((int)blockIdx.x < tab_blocks + zero_blocks) {
    const int64_t z = t - (int64_t)tab_blocks * 256;
    if (z < a.zero_n) a.zero[z] = 0;
    return;
  }
  const int64_t o = t - (int64_t)(tab_blocks + zero_blocks) * 256;
  if (o >= a.dst_len) return;
  const int64_t i = a.dst_lo + o;
  float v = 0.f;
  if (i >= 0 && i < a.n) {
    // FP32 from here on: the scale is a power of two, so the product is the
    // scaled value rounded once; a sample that is not finite in FP32 is flagged
    v = (float)((const TI *)a.src)[i] * a.scale;
    if (!isfinite(v)) {
      __hip_atomic_store(a.bad, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      v = 0.f;
    }
  }
  a.dst[o] = v;
}

// d[k] = sum_{|n| <= 32} g[n] u[2k - n]; g is zero at even n != 0 and 1/2 at 0,
// so the sum runs over the centre and symmetric odd pairs.  Up to
// kDecimGroup levels in one launch: a workgroup owns a run of samples of the
// deepest level and the samples over them at the levels between, loads the
// finer level's samples those need into LDS (32 more on each side per level)
// and cascades there, recomputing the halos (at four levels of 4096-sample runs
// 18 % more sums, 23 % more samples read).  A launch per level cost four launches and their gaps:
// 38.5 us of kernels for 1024 s at 2048 Hz against 21, 12 against 8.5 us for 8 s.
constexpr int kDecimSpan = 4096;                            // finer-level samples a workgroup owns at most
constexpr int kDecimBuf = kDecimSpan + 64 * ((1 << kDecimGroup) - 1) + 64;

__global__ __launch_bounds__(256) void k_decimate(DecimArgs a) {
  __shared__ float buf[kDecimBuf + kDecimBuf / 2];
  const int K = a.n_levels;
  const int64_t own0 = (a.tile0 + blockIdx.x) * a.span;     // owned samples of the deepest level
  // range [lo, hi) needed at each level
  int64_t lo[kDecimGroup + 1], hi[kDecimGroup + 1];
#pragma unroll
  for (int k = 0; k <= kDecimGroup; ++k) lo[k] = own0, hi[k] = own0 + a.span;
#pragma unroll
  for (int k = kDecimGroup - 1; k >= 0; --k)
    if (k < K) lo[k] = 2 * lo[k + 1] - kHalfQ, hi[k] = 2 * hi[k + 1] + kHalfQ - 1;
  for (int t = threadIdx.x; t < (int)(hi[0] - lo[0]); t += 256) {
    const int64_t i = lo[0] + t - a.u_lo;
    buf[t] = (i >= 0 && i < a.u_len) ? a.u[i] : 0.f;
  }
  __syncthreads();
  float *src = buf, *dst = buf + kDecimBuf;
#pragma unroll
  for (int k = 1; k <= kDecimGroup; ++k) {
    if (k <= K) {
      const DecimLevel &lv = a.level[k - 1];
      // owned and wanted samples of this level
      const int64_t w0 = max(own0 << (K - k), lv.lo), w1 = min((own0 + a.span) << (K - k), lv.hi);
      for (int t = threadIdx.x; t < (int)(hi[k] - lo[k]); t += 256) {
        const float *c = src + kHalfQ + 2 * t;      // lo[k - 1] = 2 lo[k] - kHalfQ
        float acc = __builtin_fmaf(a.g[kHalfQ], c[0], a.g[kHalfQ + 1] * (c[-1] + c[1]));
#pragma unroll
        for (int n = 3; n <= kHalfQ; n += 2) acc = __builtin_fmaf(a.g[kHalfQ + n], c[-n] + c[n], acc);
        dst[t] = acc;
        const int64_t i = lo[k] + t;
        if (i >= w0 && i < w1) lv.d[i - lv.d_lo] = acc;
      }
      __syncthreads();
      float *x = src;
      src = dst;
      dst = x;
    }
  }
}

template <typename T>
__global__ void k_cast_f64(const double *__restrict__ src, T *__restrict__ dst, int64_t n) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) dst[t] = (T)src[t];
}

__global__ void k_fill_u8(uint8_t *p, size_t bytes) {
  size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; t < bytes; t += stride) p[t] = 0;
}

__global__ void k_sigma2(const double *__restrict__ m, int n_templates, int lsum,
                         const double *__restrict__ inv_dec, double *__restrict__ out) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_templates) return;
  const double *rc = m + (int64_t)(2 * i) * lsum;
  const double *rs = rc + lsum;
  double acc = 0.0;
  for (int c = 0; c < lsum; ++c) acc += (rc[c] * rc[c] + rs[c] * rs[c]) * inv_dec[c];
  out[i] = acc;
}

// ------------------------------------------------------------ GEMM pieces

template <typename T, int BK = kBK> struct Pitch {
  // row pitch of an LDS tile in elements: +16 bytes keeps the 16-byte fragment
  // reads of 8 consecutive rows on distinct banks; FP32 fragments are single
  // words, so one extra word per row does the same
  static constexpr int value = sizeof(T) == 4 ? BK + 1 : BK + 16 / (int)sizeof(T);
};

// Register-staged copy of a [ROWS][BK] chunk of a row-major matrix through a
// buffer resource: setup() fixes each thread's byte offsets, load(k0) issues
// the 16-byte global reads for columns [k0, k0 + BK) (rows past the resource
// read as zero), store() writes them to LDS.
template <typename T, int ROWS, int BK = kBK, int THREADS = kThreads> struct ChunkLoader {
  static constexpr int EPV = 16 / (int)sizeof(T);   // elements per 16-byte vector
  static constexpr int VPR = BK / EPV;               // vectors per row
  static constexpr int NV = ROWS * VPR;
  static constexpr int PER = (NV + THREADS - 1) / THREADS;
  uint4 r[PER];
  int voff[PER];

  __device__ __forceinline__ void setup(int ld) {
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int v = threadIdx.x + p * THREADS;
      voff[p] = v < NV ? ((v / VPR) * ld + (v % VPR) * EPV) * (int)sizeof(T) : 0x7ffffff0;
    }
  }
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, int soff_bytes) {
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, voff[p], soff_bytes, 0);
      r[p] = make_uint4(v[0], v[1], v[2], v[3]);
    }
  }
  __device__ __forceinline__ void store(T *lds) const {
    constexpr int P = Pitch<T, BK>::value;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int v = threadIdx.x + p * THREADS;
      if (NV % THREADS != 0 && v >= NV) break;
      const int row = v / VPR, c = v % VPR;
      if constexpr (sizeof(T) == 4) {
        float *d = (float *)lds + row * P + c * 4;
        d[0] = __uint_as_float(r[p].x);
        d[1] = __uint_as_float(r[p].y);
        d[2] = __uint_as_float(r[p].z);
        d[3] = __uint_as_float(r[p].w);
      } else {
        *(uint4 *)(lds + row * P + c * EPV) = r[p];
      }
    }
  }
};

// ---------------------------------------------------------------- FIR
// o[l, k] = sum_m U[l, m] x[k - J/D - m] as D = A B with A = taps reversed
// (Ar[l, m'] = U[l, N-1-m']) and the Hankel operand B[m', k] = x[k + m' + base],
// base = -(J/D + N - 1).  The four waves share the basis rows of the
// workgroup and split its columns.  The strain window of kFirKSup taps sits
// in LDS as VEC copies shifted by 0..VEC-1 samples, so every lane's VEC
// consecutive samples are one aligned read whatever its column; the basis
// streams through double-buffered LDS with the next chunk's global reads in
// flight during the current chunk's MFMAs.
// HR (16-bit operands): the Hankel operand repeats itself shifted, so the
// fragment of column block nt at k-step g is that of block 0 at k-step
// g + 2 nt (32 columns = 2 k-steps of 16 taps).  Each wave then keeps, per
// k-step parity, a window of NT fragments in registers and reads one new
// fragment from LDS per k-step instead of NT.
// N strain samples from index i of the level (out of range: zero), all reads
// in flight at once.
template <int N>
__device__ __forceinline__ void fir_window_read(__amdgpu_buffer_rsrc_t rx, int64_t i, int64_t x_len, float (&v)[N]) {
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int off = (i + u >= 0 && i + u < x_len) ? (int)(i + u) * 4 : -4;
    v[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, off, 0, 0));
  }
}

// One 16-byte unit of each of the VEC shifted copies (copy r starts at r WC):
// v[r ..] from position `at`.
template <typename T, int WC, int N> __device__ __forceinline__ void fir_window_write(T *at, const float (&v)[N]) {
  constexpr int G = 16 / (int)sizeof(T);
#pragma unroll
  for (int r = 0; r < Op<T>::VEC; ++r) {
    T h[G];
#pragma unroll
    for (int g = 0; g < G; ++g) h[g] = Op<T>::cvt(v[r + g]);
    *(uint4 *)(at + r * WC) = __builtin_bit_cast(uint4, h);
  }
}

// Output of one wave: basis rows from rbeg, columns from cbeg.  A lane holds
// column cbeg + 32 nt + lane % 32, rows rb..rb+3 for each group of four; level-0
// slices write the time-major operand, lower-rate slices a channel-major
// buffer for the interpolation (FP32 when the operand type is BF16).
template <typename T, int MT, int NT>
__device__ __forceinline__ void fir_store(const FirJob &jb, const f32x16 (&acc)[MT][NT], int rbeg, int64_t cbeg) {
  typedef Op<T> O;
  const int lane = threadIdx.x & 63;
  const int col_limit = jb.col_limit, ldo = jb.ldo;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int64_t col = cbeg + nt * 32 + (lane & 31);
    if (col >= jb.k_hi) continue;
    const int64_t ro = (col - jb.out_lo) * (int64_t)ldo + jb.col0;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int rb = rbeg + mt * 32 + 8 * g + 4 * (lane >> 5);
        if (rb + 4 <= col_limit) {
          if (jb.out_cm && jb.out_f32) {
            float *o = (float *)jb.out + (col - jb.out_lo);
#pragma unroll
            for (int q = 0; q < 4; ++q) o[(int64_t)(rb + q) * ldo] = acc[mt][nt][4 * g + q];
          } else if (jb.out_cm) {
            T *o = (T *)jb.out + (col - jb.out_lo);
#pragma unroll
            for (int q = 0; q < 4; ++q) o[(int64_t)(rb + q) * ldo] = O::cvt(acc[mt][nt][4 * g + q]);
          } else if (jb.out_f32) {
            float *o = (float *)jb.out + ro + rb;
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = acc[mt][nt][4 * g + q];
          } else {
            T *o = (T *)jb.out + ro + rb;
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = O::cvt(acc[mt][nt][4 * g + q]);
          }
        }
      }
  }
}

// WM x WN waves, each 32 MT basis rows x 32 NT columns.
template <typename T, int MT, int NT, int WM, int WN, int BK, bool HR> struct FirTile {
  typedef Op<T> O;
  static_assert(!HR || O::KS == 16, "the fragment window needs 16 taps per k-step");
  static constexpr int THREADS = 64 * WM * WN;
  static constexpr int BM = 32 * MT * WM, BN = 32 * NT * WN;
  static constexpr int P = Pitch<T, BK>::value;
  // strain window: BN columns + kFirKSup taps (+ the fragments the HR window
  // reads ahead past its last k-step).  With 16-bit operands the copies are
  // padded to WC = 32 mod 64 elements: the 16-byte fragment reads, each lane
  // in its own copy, then run without LDS bank conflicts (the bank-conflict
  // counter reads zero there; at 0, 16, 40 and 48 mod 64 it does not)
  static constexpr int WC0 = BN + kFirKSup + 16 + (HR ? 2 * NT * 16 : 0);
  static constexpr int WC = O::VEC == 8 ? (WC0 + 31) / 64 * 64 + 32 : WC0;
  static constexpr int A_BYTES = (BM * P * (int)sizeof(T) + 15) / 16 * 16;   // one basis chunk
  static constexpr int LDS = 2 * A_BYTES + O::VEC * WC * (int)sizeof(T);

  static __device__ __forceinline__ void run(const FirJob &jb, int64_t li, char *lds);
};

template <typename T, int MT, int NT, int WM, int WN, int BK, bool HR>
__device__ __forceinline__ void FirTile<T, MT, NT, WM, WN, BK, HR>::run(const FirJob &jb, int64_t li, char *lds) {
  T *const Bc = (T *)(lds + 2 * A_BYTES);
  const int rows = jb.rows, np = jb.np;
  const T *a = (const T *)jb.basis;
  const int lane = threadIdx.x & 63;
  const int wm = (threadIdx.x >> 6) / WN, wn = (threadIdx.x >> 6) % WN;
  const int64_t r0 = (li % jb.n_rtiles) * BM;
  const int64_t i0 = jb.k_lo + (li / jb.n_rtiles) * BN;

  f32x16 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[mt][nt][e] = 0.f;

  // basis rows [r0, rows) of this workgroup; strain samples [0, x_len)
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(a + r0 * np, (rows - r0) * (int64_t)np * (int64_t)sizeof(T));
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(jb.x, jb.x_len * 4);
  const int64_t x_len = jb.x_len;
  ChunkLoader<T, BM, BK, THREADS> la;
  la.setup(np);
  la.load(ra, 0);
  // np is a multiple of kBK; with BK = 2 kBK the last chunk may hold one
  // valid half (the k-steps past np are skipped, whatever the loads brought)
  const int nchunks = (np + BK - 1) / BK;
  // lane's shifted copy: its column offset within a fragment is constant mod VEC
  const int lr = (lane & 31) % O::VEC;
  const T *bl = Bc + lr * WC + (wn * NT * 32 + (lane & 31) + (lane >> 5) * O::VEC - lr);
  // 32-column fragments of this wave that start before k_hi: a wave wholly
  // past the end of a ragged last tile skips its MFMAs (it still loads and
  // syncs); the HR window needs all NT fragments, so a partly live wave takes
  // the plain k-steps
  const int64_t wcol = i0 + wn * NT * 32;
  const int live = (int)(jb.k_hi <= wcol ? 0 : std::min<int64_t>(NT, (jb.k_hi - wcol + 31) / 32));
  int ksup = 0;
  typename O::vec hw[2][HR ? NT : 1];   // HR: fragment windows of the even and odd k-steps
  for (int c = 0; c < nchunks; ++c) {
    const int kc = c * BK;
    T *const at = (T *)(lds + (c & 1) * A_BYTES);
    if (kc % kFirKSup == 0) {
      // new strain window for taps [kc, kc + kFirKSup); out-of-range samples read as zero
      if (c > 0) __syncthreads();
      ksup = kc;
      // copy r holds x[w0 + t + r] at t: a thread takes G consecutive
      // positions of every copy, issues the G + VEC - 1 sample reads it needs
      // back to back, and writes each copy's G values as one 16-byte store
      const int64_t w0 = i0 + kc + jb.base - jb.x_lo;
      constexpr int G = 16 / (int)sizeof(T);
      static_assert(WC % G == 0, "the strain window is whole 16-byte units");
      for (int t0 = threadIdx.x * G; t0 < WC; t0 += THREADS * G) {
        float v[G + O::VEC - 1];
        fir_window_read<G + O::VEC - 1>(rx, w0 + t0, x_len, v);
        fir_window_write<T, WC>(Bc + t0, v);
      }
    }
    la.store(at);
    __syncthreads();
    if (c + 1 < nchunks) la.load(ra, (kc + BK) * (int)sizeof(T));
    auto ksteps = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int ks = 0; ks < BK / O::KS; ++ks) {
        if (BK > kBK && kc + ks * O::KS >= np) break;
        typename O::vec af[MT], bf[NT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          af[mt] = *(const typename O::vec *)(at + (wm * 32 * MT + mt * 32 + (lane & 31)) * P + ks * O::KS +
                                             (lane >> 5) * O::VEC);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) bf[nt] = *(const typename O::vec *)(bl + (kc - ksup) + nt * 32 + ks * O::KS);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = O::mfma(af[mt], bf[nt], acc[mt][nt]);
      }
    };
    if constexpr (HR) {
      if (live == NT) {
        // F(j): block-0 fragment j k-steps into the strain window
        auto F = [&](int j) __attribute__((always_inline)) {
          return *(const typename O::vec *)(bl + j * O::KS);
        };
        const int g0 = (kc - ksup) / O::KS;
        if (kc == ksup) {
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            hw[0][nt] = F(2 * nt);
            hw[1][nt] = F(1 + 2 * nt);
          }
        }
#pragma unroll
        for (int ks = 0; ks < BK / O::KS; ++ks) {
          if (BK > kBK && kc + ks * O::KS >= np) break;
          typename O::vec af[MT];
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            af[mt] = *(const typename O::vec *)(at + (wm * 32 * MT + mt * 32 + (lane & 31)) * P + ks * O::KS +
                                               (lane >> 5) * O::VEC);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = O::mfma(af[mt], hw[ks & 1][nt], acc[mt][nt]);
          // this parity's next k-step (g + 2) needs blocks shifted by one
#pragma unroll
          for (int nt = 0; nt + 1 < NT; ++nt) hw[ks & 1][nt] = hw[ks & 1][nt + 1];
          hw[ks & 1][NT - 1] = F(g0 + ks + 2 * NT);
        }
      } else if (live > 0) {
        ksteps();
      }
    } else {
      if (live > 0) ksteps();
    }
  }

  fir_store<T, MT, NT>(jb, acc, (int)r0 + wm * 32 * MT, i0 + wn * NT * 32);
}

// Narrow tile of 16-bit operands: 64 basis rows x 128 columns, 2 x 2 waves of
// 32 x 64 with the Hankel fragment window.  It is for deep filters with few
// columns, where a CU has little work at a time and the basis comes from
// memory: a chunk of 64 taps is 256 cycles of MFMAs per wave against a read
// latency of some 2000, so the chunks go straight into a ring of kRing LDS
// buffers, six ahead (rows of 128 bytes, 16-byte chunks swizzled as in the
// mixing kernel), and a window's strain reads go out a chunk early.
// FIR of an 8 s block of 1024 templates 52 -> 34 us, of a serving tick of 12
// banks 57 -> 38 us, of the 64-template single-rate call 18 -> 12 us; the same
// tile with the wide one's register-staged chunks took 41 us on the first.
// Fragment reads of 1 KB per MFMA bound it where it fills a CU (the wide tile
// reads 0.4 KB), so a full chip keeps the wide tile.
template <typename T> struct FirNarrow16 {
  typedef Op<T> O;
  typedef typename O::vec vec;
  static constexpr int BM = 64, BN = 128, BK = 64, NT = 2, kRing = 7;
  static constexpr int THREADS = 256;
  static constexpr int WC0 = BN + kFirKSup + 16 + 2 * NT * 16;
  static constexpr int WC = (WC0 + 31) / 64 * 64 + 32;
  static constexpr int CHUNK = BM * BK * 2;
  static constexpr int LDS = kRing * CHUNK + 8 * WC * 2;
  static_assert(WC >= WC0 && WC % 8 == 0 && WC <= THREADS * 8, "one 16-byte unit of the window per thread at most");
  static_assert(kFirKSup % BK == 0, "whole chunks per strain window");

  static __device__ __forceinline__ void run(const FirJob &jb, int64_t li, char *lds) {
    typedef __attribute__((address_space(3))) void lds_ptr;
    T *const Bc = (T *)(lds + kRing * CHUNK);
    const int rows = jb.rows, np = jb.np;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int64_t r0 = (li % jb.n_rtiles) * BM;
    const int64_t i0 = jb.k_lo + (li / jb.n_rtiles) * BN;
    const __amdgpu_buffer_rsrc_t ra =
        make_rsrc((const T *)jb.basis + r0 * np, (rows - r0) * (int64_t)np * (int64_t)sizeof(T));
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(jb.x, jb.x_len * 4);
    const int64_t x_len = jb.x_len;
    const int nchunks = (np + BK - 1) / BK;
    // load j of a chunk: rows 32 j + 8 wave .. + 7, lane's 16 bytes at position lane % 8 of its row
    const int vrow = 8 * wave + (lane >> 3);
    const int vo = vrow * np * 2 + ((lane & 7) ^ ((vrow >> 1) & 7)) * 16;
    auto issue = [&](int c) __attribute__((always_inline)) {
      char *buf = lds + (c % kRing) * CHUNK + wave * 1024;
      // past the last chunk: zeros into the ring, so that every step adds two loads
      const int v = c < nchunks ? vo : 0x7ff00000;
      const int so = c < nchunks ? c * BK * 2 : 0;
#pragma unroll
      for (int j = 0; j < 2; ++j)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_ptr *)(buf + j * 4096), 16, v, so + (c < nchunks ? 64 * np * j : 0),
                                                 0, 0);
    };
    f32x16 acc[1][NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[0][nt][e] = 0.f;
    const int lr = (lane & 31) % 8;
    const T *bl = Bc + lr * WC + (wn * NT * 32 + (lane & 31) + (lane >> 5) * 8 - lr);
    const int fr = wm * 32 + (lane & 31), fq = lane >> 5, fs = (fr >> 1) & 7;
    const bool live = i0 + wn * NT * 32 < jb.k_hi;   // a wave past a ragged end loads and syncs only
    const int t0 = threadIdx.x * 8;
    const int64_t xw = i0 + jb.base - jb.x_lo + t0;
    float xv[15];
    if (t0 < WC) fir_window_read<15>(rx, xw, x_len, xv);
#pragma unroll
    for (int c = 0; c < kRing - 1; ++c) issue(c);
    vec hw[2][NT];
    for (int c = 0; c < nchunks; ++c) {
      const int kc = c * BK, kw = kc % kFirKSup;
      if (kw == 0) {
        if (c > 0) __syncthreads();   // the window's last reads are done
        if (t0 < WC) fir_window_write<T, WC>(Bc + t0, xv);
      }
      // this wave's part of chunk c is in (vmcnt) and its LDS accesses are done
      // (lgkmcnt); then every wave's, and chunk c - 1's buffer is free.  Not
      // __syncthreads, which would wait for the whole ring.
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(0x0070 | (2 * (kRing - 2)));
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      issue(c + kRing - 1);
      if (kw + BK == kFirKSup && c + 1 < nchunks && t0 < WC) fir_window_read<15>(rx, xw + kc + BK, x_len, xv);
      if (!live) continue;
      const char *at = lds + (c % kRing) * CHUNK + fr * 128;
      auto F = [&](int j) __attribute__((always_inline)) { return *(const vec *)(bl + j * 16); };
      if (kw == 0) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          hw[0][nt] = F(2 * nt);
          hw[1][nt] = F(1 + 2 * nt);
        }
      }
      // the chunk's fragments are all read before its products (one LDS latency
      // per chunk, not per k-step)
      vec af[BK / 16], nx[BK / 16];
#pragma unroll
      for (int ks = 0; ks < BK / 16; ++ks) {
        af[ks] = *(const vec *)(at + ((2 * ks + fq) ^ fs) * 16);
        nx[ks] = F(kw / 16 + ks + 2 * NT);
      }
      __builtin_amdgcn_sched_barrier(0);
      auto kstep = [&](int ks) __attribute__((always_inline)) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[0][nt] = O::mfma(af[ks], hw[ks & 1][nt], acc[0][nt]);
        hw[ks & 1][0] = hw[ks & 1][1];
        hw[ks & 1][1] = nx[ks];
      };
      kstep(0);
      kstep(1);
      if (kc + 32 < np) {   // np is a multiple of 32: the last chunk may hold half
        kstep(2);
        kstep(3);
      }
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);   // the zeros past the last chunk have landed
    fir_store<T, 1, NT>(jb, acc, (int)r0 + wm * 32, i0 + wn * NT * 32);
  }
};

// A launch of one tile shape, or (narrow jobs) of two: the same threads, the
// narrow tile's 64 rows x 128 columns.
constexpr int kFirNarrowBM = 64, kFirNarrowBN = 128;
template <typename T> struct FirNarrow { typedef FirNarrow16<T> tile; };
template <> struct FirNarrow<float> { typedef FirTile<float, 1, 1, 2, 4, kBK, false> tile; };   // waves of 32 x 32

template <typename T, int MT, int NT, int NW, int BK, bool HR, bool NARROW>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 2 : 1) void k_fir(const FirJob *__restrict__ jobs, int n_jobs) {
  typedef FirTile<T, MT, NT, 1, NW, BK, HR> Wide;
  typedef typename FirNarrow<T>::tile Narrow;
  static_assert(!NARROW || (Narrow::THREADS == Wide::THREADS && Narrow::BM == kFirNarrowBM && Narrow::BN == kFirNarrowBN),
                "one launch of both shapes");
  __shared__ __attribute__((aligned(1024))) char lds[NARROW && Narrow::LDS > Wide::LDS ? Narrow::LDS : Wide::LDS];
  const FirJob &jb = jobs[find_job(jobs, n_jobs, blockIdx.x)];
  const int64_t li = (int64_t)blockIdx.x - jb.item0;
  if constexpr (NARROW) {
    if (jb.narrow) return Narrow::run(jb, li, lds);
  }
  Wide::run(jb, li, lds);
}

// ----------------------------------------------------- interpolation on MFMA
// One or two half-band x2 stages as one composite filter h_R (R = 2 or 4):
// out[c][n] = sum_u src[c][u] h_R[n - R u].  For a 32-sample output tile at n0
// (a multiple of 32) the taps that matter are u = U0 + kk, kk < 64, with
// U0 = n0 / R - (32 - 32 / R), and H[kk][t] = h_R[t - R kk + 32 R - 32] is the
// same matrix for every tile: it stays in registers as MFMA fragments while
// the channel-major source rows stream in.  A hop into a channel-major buffer
// computes D[c][t] (source rows as the A operand); the last hop, into the
// time-major mixing operand, computes D[t][c] with the operands swapped, so
// each store instruction writes 32 consecutive channels of two samples.
// TS: source and low-rate buffer type; TD: operand type of the last hop.
// What bounds it: long blocks the writes of the operand (1024 s of 1024
// templates: 1.14 GB in 503 us, 2.3 TB/s; a large copy writes at 2.5), ones
// that stay in the caches latency and the address units.  Each wave therefore
// brings its 32 source rows' windows to LDS with coalesced direct loads (read
// from memory as fragments, every lane's 16 bytes were a line of their own, and each
// block was read twice: 59 against 82 us for FP32, 48 s), works tile by tile, so
// that a tile's stores go out while the next is computed (few registers: with
// 16-bit sources five or six waves per SIMD; FP32 sources' windows leave LDS for
// two or three), writes 32-column blocks that start at the operand's own 32-column grid
// with a dword per lane, without bounds checks inside, and the tasks run over
// all slices' blocks of a column tile.  Before and after: FP32, 48 s 109 -> 59 us;
// FP16, 48 s with the series 37 -> 22, 8 s 17 -> 13, 1024 s 630 -> 554; BF16, 200 s
// 174 -> 131.  Tasks of 64 columns (whole lines per store): 1024 s 496, but 48 s 29
// and 8 s 17 us.  Neither a row pitch of an odd number of lines nor
// non-temporal stores changed the long blocks.
//
// A lane's source window: the fragment of tile t at k-step ks is the
// VEC-sample block 2 ks + SB t past the lane's first one (the tiles' source
// windows start 32 / R = SB VEC samples apart), so a lane reads each block that
// the MFMAs use once, all reads issued before the MFMAs.  With SB even only the
// even blocks are used.
//
// FP32 sources of the BF16 operand path (SPLIT): every source value x and filter
// tap h is split into a BF16 pair, x = x_hi + x_lo with x_hi = bf16(x) and
// x_lo = bf16(x - x_hi) (16 significant bits), and a product takes three
// BF16 MFMAs, x_hi h_hi + x_lo h_hi + x_hi h_lo (the dropped x_lo h_lo and
// the splits' remainders are of order 2^-16 relative), with FP32 sums: the
// 32x32x16 instruction in place of eight FP32 32x32x2 ones per k-step.
// Blocks are 8 source samples (two 16-byte reads), laid out as for 16-bit
// sources; hf holds the filter's hi fragments, then its lo fragments.
// 16-byte units of a source row's window of a wave task (64 samples for the
// first tile, 32 / R more for each further one), odd for FP32 rows (LDS banks).
template <typename TS> __host__ __device__ constexpr int up_units(int R) {
  const int u = (64 + (kUpCols - 32) / R) * (int)sizeof(TS) / 16;
  return sizeof(TS) == 4 ? u | 1 : u;
}

// LDS of a wave whose hops' factors are r_min or more, in whole 64-unit loads.
template <typename TS> __host__ __device__ constexpr int up_wave_lds(int r_min) {
  return (32 * up_units<TS>(r_min) + 63) / 64 * 1024;
}

template <typename TS, bool SPLIT> struct UpWindow {
  typedef Op<TS> O;
  typedef typename O::vec vec;
  static_assert(O::KS == 2 * O::VEC, "two VEC blocks per k-step");
  static constexpr int VEC = O::VEC, NKS = 64 / O::KS, SB4 = 8 / VEC;   // SB for R = 4; twice that for R = 2
  static constexpr int NB = 2 * (NKS - 1) + 2 * SB4 * (kUpCols / 32 - 1) + 1;
  vec blk[NB];

  // row: the lane's row in LDS, at the lane's first block
  template <int SB> __device__ __forceinline__ void read(const char *row) {
#pragma unroll
    for (int j = 0; j <= 2 * (NKS - 1) + SB * (kUpCols / 32 - 1); ++j) {
      if (SB % 2 == 0 && (j & 1)) continue;
      blk[j] = *(const vec *)(row + j * (int)sizeof(vec));
    }
  }
  template <bool TM, int SB> __device__ __forceinline__ f32x16 tile(int t, const vec *hf, const vec *) const {
    f32x16 acc = {};
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const vec a = blk[2 * ks + SB * t];
      acc = TM ? O::mfma(hf[ks], a, acc) : O::mfma(a, hf[ks], acc);
    }
    return acc;
  }
};

struct uint4x2 {
  __attribute__((ext_vector_type(4))) unsigned int a, b;
};

template <> struct UpWindow<float, true> {
  typedef Op<__bf16> O;
  typedef bf16x8 vec;
  typedef float f32x8 __attribute__((ext_vector_type(8)));
  static constexpr int VEC = 8, NKS = 4, SB4 = 1;
  static constexpr int NB = 2 * (NKS - 1) + 2 * SB4 * (kUpCols / 32 - 1) + 1;
  vec hi[NB], lo[NB];

  template <int SB> __device__ __forceinline__ void read(const char *row) {
#pragma unroll
    for (int j = 0; j <= 2 * (NKS - 1) + SB * (kUpCols / 32 - 1); ++j) {
      if (SB % 2 == 0 && (j & 1)) continue;
      const uint4x2 v = {*(const decltype(uint4x2::a) *)(row + j * 32), *(const decltype(uint4x2::a) *)(row + j * 32 + 16)};
      const f32x8 x = __builtin_bit_cast(f32x8, v);
      __bf16 h[8], l[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        h[e] = (__bf16)x[e];
        l[e] = (__bf16)(x[e] - (float)h[e]);
      }
      hi[j] = __builtin_bit_cast(vec, h);
      lo[j] = __builtin_bit_cast(vec, l);
    }
  }
  template <bool TM, int SB> __device__ __forceinline__ f32x16 tile(int t, const vec *hhi, const vec *hlo) const {
    f32x16 acc = {};
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int j = 2 * ks + SB * t;
      if (TM) {
        acc = O::mfma(hlo[ks], hi[j], acc);
        acc = O::mfma(hhi[ks], lo[j], acc);
        acc = O::mfma(hhi[ks], hi[j], acc);
      } else {
        acc = O::mfma(hi[j], hlo[ks], acc);
        acc = O::mfma(lo[j], hhi[ks], acc);
        acc = O::mfma(hi[j], hhi[ks], acc);
      }
    }
    return acc;
  }
};

// One wave task, 32 channels from r0, SB the window step of the hop's factor.
// TM false: into a channel-major buffer.  TM true: the last hop, into a
// 32-column block of the time-major operand (r0 below 0 where the block begins in
// the slice before; rows outside the slice are not read).  A lane then holds
// samples n0 + 32 t + 8 g + 4 (lane / 32) + q of its channel; with 16-bit operands
// two samples of neighbouring channels change hands, so that it stores a dword
// of two columns (two neighbours are both in or both out: offsets and counts of
// channels are multiples of 16).
template <typename TS, typename TD, bool TM, int SB>
__device__ __forceinline__ void upsample_task(const UpJob &jb, char *lds, int lane, int r0, int64_t n0) {
  constexpr bool SPLIT = std::is_same<TS, float>::value && std::is_same<TD, __bf16>::value;
  typedef UpWindow<TS, SPLIT> W;
  typedef typename W::vec vec;
  constexpr int CT = kUpCols / 32;
  constexpr int R = SB == W::SB4 ? 4 : 2, cR = 32 - 32 / R;
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(jb.src, jb.src_bytes);
  vec hf[W::NKS], hlo[SPLIT ? W::NKS : 1];
#pragma unroll
  for (int ks = 0; ks < W::NKS; ++ks) {
    hf[ks] = *(const vec *)((const char *)jb.hf + (ks * 64 + lane) * sizeof(vec));
    if constexpr (SPLIT) hlo[ks] = *(const vec *)((const __bf16 *)jb.hf + kInterpFragEntries + (ks * 64 + lane) * 8);
  }
  const int c = r0 + (lane & 31);
  const bool in = c >= 0 && c < jb.channels;
  {
    typedef __attribute__((address_space(3))) void lds_ptr;
    constexpr int NU = up_units<TS>(R), LOADS = (32 * NU + 63) / 64;
    const int64_t col = n0 / R - cR - jb.src_lo;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int u = i * 64 + lane, row = u / NU, k = u - row * NU, ch = r0 + row;
      const bool ok = row < 32 && ch >= 0 && ch < jb.channels;
      const int off = ok ? (int)((ch * (int64_t)jb.ld_src + col) * (int64_t)sizeof(TS)) + k * 16 : -16;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr *)(lds + i * 1024), 16, off, 0, 0, 0);
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0f70);
    asm volatile("" ::: "memory");
  }
  W w;
  w.template read<SB>(lds + (lane & 31) * up_units<TS>(R) * 16 + (lane >> 5) * (int)(W::VEC * sizeof(TS)));
  if constexpr (TM) {
    const int ld = jb.ld_dst * (int)sizeof(TD);
    const bool whole = n0 >= jb.n_lo && n0 + kUpCols <= jb.n_hi;   // all but the ends: no checks, 32-bit offsets
    const __amdgpu_buffer_rsrc_t rd =
        make_rsrc((TD *)jb.dst + (n0 - jb.dst_abs0) * jb.ld_dst, whole ? (int64_t)kUpCols * ld : 0);
    // 16 bits: of samples q and q + 1 (q even) the even lane stores the first for both channels, the odd lane the second
    const int odd = sizeof(TD) == 2 ? lane & 1 : 0;
    const uint32_t sel = odd ? 0x07060302u : 0x01000504u;
    const int vo = in ? (jb.col0 + c - odd) * (int)sizeof(TD) + (4 * (lane >> 5) + odd) * ld : 0x7ff00000;
    auto put = [&](uint32_t v, int t, int e) __attribute__((always_inline)) {
      if (whole) {
        __builtin_amdgcn_raw_buffer_store_b32(v, rd, vo, (32 * t + 8 * (e >> 2) + (e & 3)) * ld, 0);
      } else if (in) {
        const int64_t n = n0 + 32 * t + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3) + odd;
        if (n >= jb.n_lo && n < jb.n_hi)
          *(uint32_t *)((TD *)jb.dst + (n - jb.dst_abs0) * jb.ld_dst + jb.col0 + c - odd) = v;
      }
    };
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const f32x16 acc = w.template tile<TM, SB>(t, hf, hlo);
      if constexpr (sizeof(TD) == 4) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float v = acc[e];
          put(__builtin_bit_cast(uint32_t, v), t, e);
        }
      } else {
        typedef TD pair __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
          const pair p = {Op<TD>::cvt(acc[e]), Op<TD>::cvt(acc[e + 1])};
          const uint32_t own = __builtin_bit_cast(uint32_t, p);
          const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)own, 0xB1, 0xf, 0xf, true);
          put(__builtin_amdgcn_perm(own, other, sel), t, e);
        }
      }
      __builtin_amdgcn_sched_barrier(0);   // a tile's stores go out before the next tile's results take registers
    }
  } else {
    // lane holds sample n0 + 32 t + lane % 32 of channels r0 + 8 g + 4 (lane / 32) + q;
    // channels is a multiple of 16, so a lane's four channels are all in or all out
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const f32x16 acc = w.template tile<TM, SB>(t, hf, hlo);
      const int64_t n = n0 + 32 * t + (lane & 31);
      if (n >= jb.n_lo && n < jb.n_hi) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int rb = r0 + 8 * g + 4 * (lane >> 5);
          if (rb >= jb.channels) continue;
          TS *d = (TS *)jb.dst + (int64_t)rb * jb.ld_dst + (n - jb.dst_abs0);
#pragma unroll
          for (int q = 0; q < 4; ++q) d[(int64_t)q * jb.ld_dst] = Op<TS>::cvt(acc[4 * g + q]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <typename TS, typename TD>
__global__ __launch_bounds__(256) void k_upsample(const UpJob *__restrict__ jobs, int n_jobs, int r_min) {
  const int last = find_job(jobs, n_jobs, blockIdx.x);   // the last job of the items' group
  // The 8 XCDs take workgroups round-robin and every group's items start at a
  // multiple of 8: give each XCD one contiguous run of the group's tasks, so
  // neighbouring column tiles (whose source windows overlap) share one L2.
  const int rtiles = jobs[last].grp_rtiles;
  const int64_t n_tasks = (int64_t)rtiles * jobs[last].n_ctiles;
  const int64_t per_xcd = (n_tasks + 31) / 32;          // items per XCD, 4 tasks each
  const int64_t b = (int64_t)blockIdx.x - jobs[last].item0;
  const int64_t li = (b & 7) * per_xcd + (b >> 3);
  const int lane = threadIdx.x & 63;
  // wave task: a block of channels x kUpCols output samples
  const int64_t task = li * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (task >= n_tasks) return;
  int rt = (int)(task % rtiles), k = last;
  while (jobs[k].rt0 > rt) --k;
  const UpJob &jb = jobs[k];
  rt -= jb.rt0;
  const int64_t n0 = jb.n_first + (task / rtiles) * kUpCols;
  extern __shared__ __attribute__((aligned(1024))) char lds_all[];
  char *const lds = lds_all + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * up_wave_lds<TS>(r_min);
  constexpr int SB4 = UpWindow<TS, std::is_same<TS, float>::value && std::is_same<TD, __bf16>::value>::SB4;
  if (jb.dst_tm) {
    const int r0 = rt * 32 - jb.col0 % 32;
    if (jb.r == 4) upsample_task<TS, TD, true, SB4>(jb, lds, lane, r0, n0);
    else upsample_task<TS, TD, true, 2 * SB4>(jb, lds, lane, r0, n0);
  } else if (jb.r == 4) {
    upsample_task<TS, TD, false, SB4>(jb, lds, lane, rt * 32, n0);
  } else {
    upsample_task<TS, TD, false, 2 * SB4>(jb, lds, lane, rt * 32, n0);
  }
}

// ------------------------------------------------------- mixing + peaks
// Y[c, n] = sum_k M[c, k] O[n, k] over the concatenated basis; rows 2i and
// 2i+1 (cos, sin) of template i land in the same lane, so |z|^2 and the
// running per-template peak (value, sample) stay in registers.  One
// workgroup owns whole trigger windows of one row tile: the peak of a
// window is reduced across lanes and waves without atomics (larger |z|^2
// first, then lower sample).  The phase at the peak is recomputed by
// k_peak_phase from the same operands.
__device__ __forceinline__ bool better(float va, int na, float vb, int nb) {
  return va > vb || (va == vb && na < nb);
}

// Row tile, window (within the job) and part of the window of workgroup b of
// a job.  A window's column steps are shared by jb.parts workgroups, each a
// run of them.  XCD-aware order: the 8 XCDs take workgroups round-robin
// (every job's items start at a multiple of 8), so all row tiles of one
// (window, part) unit get the same XCD and neighbouring slots (shared operand
// rows in that XCD's L2).  A job of fewer than 8 units would leave XCDs idle
// that way: its items run unit-major over the row tiles instead, spread over
// all XCDs.
struct MixUnit {
  int rt, part;
  int64_t wl;
};

__device__ __forceinline__ MixUnit mix_unit(const MixJob &jb, int64_t b) {
  MixUnit m;
  int64_t u;
  if (jb.nw * jb.parts >= 8) {
    const int64_t slot = b >> 3;
    m.rt = (int)(slot % jb.n_rtiles);
    u = (slot / jb.n_rtiles) * 8 + (b & 7);
  } else {
    m.rt = (int)(b % jb.n_rtiles);
    u = b / jb.n_rtiles;
  }
  m.wl = u / jb.parts;
  m.part = (int)(u - m.wl * jb.parts);
  return m;
}

template <typename T, int MT, int NT, int WM, int WN, int BK, bool SNR>
__global__ __launch_bounds__(64 * WM * WN) void k_mix_peak(const MixJob *__restrict__ jobs, int n_jobs) {
  typedef Op<T> O;
  constexpr int THREADS = 64 * WM * WN;
  constexpr int BM = 32 * MT * WM, BN = 32 * NT * WN;
  constexpr int P = Pitch<T, BK>::value;
  __shared__ __attribute__((aligned(16))) T As[2][BM * P];
  __shared__ __attribute__((aligned(16))) T Bs[2][BN * P];
  __shared__ VN red[WN][BM / 2];

  const MixJob &jb = jobs[find_job(jobs, n_jobs, blockIdx.x)];
  const int64_t b = (int64_t)blockIdx.x - jb.item0;
  const MixUnit un = mix_unit(jb, b);
  if (un.wl >= jb.nw) return;
  const int rt = un.rt;
  const int64_t w = jb.w0 + un.wl;
  const T *mix = (const T *)jb.mix;
  const int rows = jb.rows, kcat = jb.kcat, kld = jb.kld, n_templates = jb.n_templates;
  const float inv_scale = jb.inv_scale;

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int64_t r0 = (int64_t)rt * BM;
  const int64_t ws = (w * jb.win_p) / jb.win_q;
  int64_t we = ((w + 1) * jb.win_p) / jb.win_q;
  if (we > jb.n_end) we = jb.n_end;
  const T *ocat = (const T *)jb.ocat + (ws - jb.ocat_abs0) * (int64_t)kld;   // row of sample ws
  VN best[MT][8];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int p = 0; p < 8; ++p) best[mt][p] = VN{-1.f, 0x7fffffff};

  // mixing rows [r0, rows) and operand rows [ws, we) of this workgroup; rows
  // past either end read as zero
  constexpr int ESZ = (int)sizeof(T);
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(mix + r0 * kld, (rows - r0) * (int64_t)kld * ESZ);
  const __amdgpu_buffer_rsrc_t rb = make_rsrc(ocat, (we - ws) * (int64_t)kld * ESZ);
  // kcat is a multiple of 32; with BK = 64 the k-steps past kcat are skipped
  // (the rows' pitch kld is a multiple of 64: the chunks stay inside a row)
  const int nchunks = (kcat + BK - 1) / BK;
  ChunkLoader<T, BM, BK, THREADS> la;
  ChunkLoader<T, BN, BK, THREADS> lb;
  la.setup(kld);
  lb.setup(kld);
  // the part's columns of the window, whole column steps
  const int64_t all_steps = (we - ws + BN - 1) / BN;
  const int64_t nbeg = ws + all_steps * un.part / jb.parts * BN;
  const int64_t nfin = min(we, ws + all_steps * (un.part + 1) / jb.parts * BN);
  if (nbeg >= nfin) return;   // a short last window has fewer steps than parts
  la.load(ra, 0);
  lb.load(rb, (int)(nbeg - ws) * kld * ESZ);
  int it = 0;  // chunk counter across column steps: LDS buffer parity
  for (int64_t n0 = nbeg; n0 < nfin; n0 += BN) {
    const int brow = (int)(n0 - ws) * kld * ESZ;   // byte offset of this step's first operand row
    f32x16 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[mt][nt][e] = 0.f;

    for (int c = 0; c < nchunks; ++c, ++it) {
      const int cur = it & 1;
      la.store(As[cur]);
      lb.store(Bs[cur]);
      __syncthreads();
      if (c + 1 < nchunks) {
        la.load(ra, (c + 1) * BK * ESZ);
        lb.load(rb, brow + (c + 1) * BK * ESZ);
      } else if (n0 + BN < nfin) {
        la.load(ra, 0);
        lb.load(rb, brow + BN * kld * ESZ);
      }
#pragma unroll
      for (int ks = 0; ks < BK / O::KS; ++ks) {
        if (BK > 32 && c * BK + ks * O::KS >= kcat) break;
        typename O::vec af[MT], bf[NT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          af[mt] = *(const typename O::vec *)(As[cur] + (wm * 32 * MT + mt * 32 + (lane & 31)) * P + ks * O::KS +
                                             (lane >> 5) * O::VEC);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          bf[nt] = *(const typename O::vec *)(Bs[cur] + (wn * 32 * NT + nt * 32 + (lane & 31)) * P + ks * O::KS +
                                             (lane >> 5) * O::VEC);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = O::mfma(af[mt], bf[nt], acc[mt][nt]);
      }
    }

    // epilogue: complex SNR of 8 templates per lane per row tile
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int64_t col = n0 + wn * 32 * NT + nt * 32 + (lane & 31);
      const bool ok = col < we;
      const int rel = (int)(col - ws);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          const float re = acc[mt][nt][2 * p], im = acc[mt][nt][2 * p + 1];
          const float v = re * re + im * im;
          if (ok && v > best[mt][p].v) best[mt][p] = VN{v, rel};
          if (SNR && ok) {
            const int64_t i = (r0 + wm * 32 * MT + mt * 32 + 8 * (p >> 1) + 4 * (lane >> 5) + 2 * (p & 1)) >> 1;
            if (i < n_templates) {
              // written once and not read here: a non-temporal store
              typedef float fv2 __attribute__((ext_vector_type(2)));
              __builtin_nontemporal_store(fv2{re * inv_scale, im * inv_scale},
                                          (fv2 *)(jb.snr + (i * jb.snr_ld + (col - jb.snr_abs0)) * 2));
            }
          }
        }
      }
    }
  }

  // reduce the 32 columns of each half-wave, then the waves that share rows
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      VN bb = best[mt][p];
#pragma unroll
      for (int off = 1; off < 32; off <<= 1) {
        const float ov = __shfl_xor(bb.v, off);
        const int on = __shfl_xor(bb.n, off);
        if (better(ov, on, bb.v, bb.n)) bb = VN{ov, on};
      }
      if ((lane & 31) == 0) red[wn][wm * 16 * MT + mt * 16 + 4 * (p >> 1) + 2 * (lane >> 5) + (p & 1)] = bb;
    }
  __syncthreads();
  for (int t = threadIdx.x; t < BM / 2; t += THREADS) {
    VN bb = red[0][t];
#pragma unroll
    for (int q = 1; q < WN; ++q)
      if (better(red[q][t].v, red[q][t].n, bb.v, bb.n)) bb = red[q][t];
    const int64_t i = r0 / 2 + t;
    if (i < n_templates) put_peak(jb, i, w, bb);
  }
}

// 16-bit operands, direct-to-LDS form of the mixing kernel.  The operand
// chunks go from global memory straight into LDS (16-byte buffer loads with
// an LDS destination: no staging registers, no LDS store instructions), two
// buffers; rows past either matrix's end read as zero.  An LDS row holds BK
// elements in 16-byte chunks, chunk q of row r at position
// q ^ ((r / (16 / CPR)) % CPR) (CPR chunks per row), so the 16 rows that 16
// lanes read in one fragment load start on distinct banks.  Each output's K
// sum runs in the same order as in k_mix_peak, so the results are
// bit-identical.  The compiled shape: 256 x 256 tiles of eight 64 x 128
// waves, K chunks of 64 (128 KiB of LDS, one workgroup per CU).  Measured and
// not kept: four 128 x 128 waves (one wave per SIMD: its 256 accumulators
// leave the epilogue spilling, 7.6 against 4.0 ms per 1024-template
// detector-call) and two independent workgroups of 128 x 256 per CU with K
// chunks of 32 (4.9 ms).
template <int BK> struct DlRow {
  static constexpr int BYTES = 2 * BK, CPR = BYTES / 16, RPI = 1024 / BYTES;   // RPI: rows per load instruction
  static __device__ __forceinline__ int swz(int row, int q) { return q ^ ((row / (16 / CPR)) % CPR); }
};

typedef __attribute__((address_space(3))) void lds_void;

// Fragments of one k-step: MT A fragments (mixing rows wm*32*MT + mt*32 +
// lane%32) and NT B fragments (operand rows wn*32*NT + nt*32 + lane%32), 8
// consecutive k values from 16 ks + 8 (lane/32).
template <typename T, int BK, int MT, int NT>
__device__ __forceinline__ void dl_frags(const char *a, const char *b, int wm, int wn, int fr, int fh, int ks,
                                         typename Op<T>::vec (&af)[MT], typename Op<T>::vec (&bf)[NT]) {
  typedef DlRow<BK> R;
  const int qc = 2 * ks + fh;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int row = wm * 32 * MT + mt * 32 + fr;
    af[mt] = *(const typename Op<T>::vec *)(a + row * R::BYTES + R::swz(row, qc) * 16);
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int row = wn * 32 * NT + nt * 32 + fr;
    bf[nt] = *(const typename Op<T>::vec *)(b + row * R::BYTES + R::swz(row, qc) * 16);
  }
}

// FIRST: the first k-step of a column step, whose accumulators start at zero
// (the zero is the MFMA's constant operand, no register clearing)
template <typename T, int MT, int NT, bool FIRST = false>
__device__ __forceinline__ void dl_mfmas(const typename Op<T>::vec (&af)[MT], const typename Op<T>::vec (&bf)[NT],
                                         f32x16 (&acc)[MT][NT]) {
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
      acc[mt][nt] = Op<T>::mfma(af[mt], bf[nt], FIRST ? f32x16{} : acc[mt][nt]);
}

// Schedule: the chunks of all column steps of the window form one sequence
// g = 0, 1, ...  (chunk c = g % nchunks of column step g / nchunks).  Within
// a chunk, the fragments of k-step ks + 1 are read while the MFMAs of ks
// run; before the MFMAs of the last k-step, every wave waits for the next
// chunk's loads and meets at the barrier, then reads the next chunk's first
// fragments and starts the loads of the chunk after it into the buffer just
// finished, and only then issues the last k-step's MFMAs.  With K chunks of
// 64 and kcat an odd multiple of 32, the last chunk of a column step holds 2
// k-steps: its upper 32 columns are loaded as out-of-range (zeros) for both
// operands, so the 4 k-steps always run and the extra products are exact
// zeros.  Waves: WM x WN, each 32 MT rows x 32 NT columns; WGS workgroups per
// CU.
template <typename T, int WM, int WN, int MT, int NT, int BK, int WGS, bool SNR>
__global__ __launch_bounds__(64 * WM * WN, WGS) void k_mix_dl(const MixJob *__restrict__ jobs, int n_jobs) {
  static_assert(sizeof(T) == 2, "16-bit operands only");
  typedef typename Op<T>::vec vec;
  typedef DlRow<BK> R;
  constexpr int NW = WM * WN, THREADS = 64 * NW;
  constexpr int BM = 32 * MT * WM, BN = 32 * NT * WN;
  constexpr int KS = BK / 16;                  // k-steps per chunk
  constexpr int JA = BM / R::RPI / NW, JB = BN / R::RPI / NW;   // load instructions per wave and chunk
  static_assert(JA * R::RPI * NW == BM && JB * R::RPI * NW == BN, "whole load instructions per wave");
  static_assert((R::RPI * NW) % 16 == 0, "one voffset per wave");
  static_assert(KS == 2 || KS == 4, "chunks of 32 or 64");
  __shared__ __attribute__((aligned(1024))) char As0[BM * R::BYTES];
  __shared__ __attribute__((aligned(1024))) char Bs0[BN * R::BYTES];
  __shared__ __attribute__((aligned(1024))) char As1[BM * R::BYTES];
  __shared__ __attribute__((aligned(1024))) char Bs1[BN * R::BYTES];
  __shared__ VN red[WN][BM / 2];

  const MixJob &jb = jobs[find_job(jobs, n_jobs, blockIdx.x)];
  const int64_t b = (int64_t)blockIdx.x - jb.item0;
  const MixUnit un = mix_unit(jb, b);
  if (un.wl >= jb.nw) return;
  const int rt = un.rt;
  const int64_t w = jb.w0 + un.wl;
  const T *mix = (const T *)jb.mix;
  const int rows = jb.rows, kcat = jb.kcat, kld = jb.kld, n_templates = jb.n_templates;
  const float inv_scale = jb.inv_scale;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int64_t r0 = (int64_t)rt * BM;
  const int64_t ws = (w * jb.win_p) / jb.win_q;
  int64_t we = ((w + 1) * jb.win_p) / jb.win_q;
  if (we > jb.n_end) we = jb.n_end;
  const T *ocat = (const T *)jb.ocat + (ws - jb.ocat_abs0) * (int64_t)kld;
  VN best[MT][8];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int p = 0; p < 8; ++p) best[mt][p] = VN{-1.f, 0x7fffffff};

  constexpr int ESZ = 2;
  // rows of pitch kld (a multiple of 64 elements: every chunk row is one
  // 128-byte line of a line-aligned row)
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(mix + r0 * kld, (rows - r0) * (int64_t)kld * ESZ);
  const __amdgpu_buffer_rsrc_t rb = make_rsrc(ocat, (we - ws) * (int64_t)kld * ESZ);
  const int nchunks = (kcat + BK - 1) / BK;
  const bool half_tail = (kcat % BK) != 0;   // K chunks of 64: the last one holds 32 columns
  // column steps [st0, st0 + nsteps) of the window are this part's
  const int all_steps = (int)((we - ws + BN - 1) / BN);
  const int st0 = all_steps * un.part / jb.parts;
  const int nsteps = all_steps * (un.part + 1) / jb.parts - st0;
  if (nsteps <= 0) return;   // a short last window has fewer steps than parts
  const int G = nsteps * nchunks;
  // Load instruction j of this wave fills LDS rows RPI (NW j + wave) .. + RPI - 1
  // of a tile, lane i the 16-byte position i % CPR of row RPI (NW j + wave) +
  // i / CPR: logical chunk swz(row, i % CPR), the same for every j (the row
  // step is a multiple of 16 rows), so one voffset serves every instruction
  // and the row step goes into the scalar offset.
  const int vrow = R::RPI * wave + lane / R::CPR;
  const int lq = R::swz(vrow, lane % R::CPR);
  const int voffs = vrow * kld * ESZ + lq * 16;
  const int voffs_tail = lq < R::CPR / 2 ? voffs : 0x7ff00000;   // upper half of a half chunk: zeros
  const int jstep = R::RPI * NW * kld * ESZ;
  auto issue = [&](int g) {
    const int c = g % nchunks, st = st0 + g / nchunks;
    const int ka = c * BK * ESZ;
    const int kb = st * BN * kld * ESZ + ka;
    const int vo = (half_tail && c == nchunks - 1) ? voffs_tail : voffs;
    char *at = (g & 1) ? As1 : As0;
    char *bt = (g & 1) ? Bs1 : Bs0;
#pragma unroll
    for (int j = 0; j < JA; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void *)(at + (NW * j + wave) * 1024), 16, vo,
                                               ka + j * jstep, 0, 0);
#pragma unroll
    for (int j = 0; j < JB; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void *)(bt + (NW * j + wave) * 1024), 16, vo,
                                               kb + j * jstep, 0, 0);
  };
  const int fr = lane & 31, fh = lane >> 5;
  vec fa0[MT], fb0[NT], fa1[MT], fb1[NT];
  issue(0);
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
  __syncthreads();
  dl_frags<T, BK, MT, NT>(As0, Bs0, wm, wn, fr, fh, 0, fa0, fb0);
  if (G > 1) issue(1);
  int g = 0;
  for (int st = 0; st < nsteps; ++st) {
    f32x16 acc[MT][NT];
    // one chunk; FIRST: the column step's first (its first k-step starts the
    // sums); skip_hi: a half chunk (its k-steps 2 and 3 are zeros: no MFMAs)
    auto chunk = [&](auto first_c, bool skip_hi) {
      constexpr bool FIRST = decltype(first_c)::value;
      const char *a = (g & 1) ? As1 : As0;
      const char *bt = (g & 1) ? Bs1 : Bs0;
      // the phases stay in this order (the scheduler would otherwise hoist
      // the barrier above the MFMAs and group the reads)
      dl_frags<T, BK, MT, NT>(a, bt, wm, wn, fr, fh, 1, fa1, fb1);
      __builtin_amdgcn_sched_barrier(0);
      dl_mfmas<T, MT, NT, FIRST>(fa0, fb0, acc);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (KS == 4) {
        dl_frags<T, BK, MT, NT>(a, bt, wm, wn, fr, fh, 2, fa0, fb0);
        __builtin_amdgcn_sched_barrier(0);
        dl_mfmas<T, MT, NT>(fa1, fb1, acc);
        __builtin_amdgcn_sched_barrier(0);
        dl_frags<T, BK, MT, NT>(a, bt, wm, wn, fr, fh, 3, fa1, fb1);
        __builtin_amdgcn_sched_barrier(0);
        if (!skip_hi) dl_mfmas<T, MT, NT>(fa0, fb0, acc);
        __builtin_amdgcn_sched_barrier(0);
      }
      // the next chunk's loads (this wave's part) are done and this wave's
      // reads of the current buffer have returned; the barrier makes both
      // hold for every wave
      __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
      __syncthreads();
      if (g + 1 < G)
        dl_frags<T, BK, MT, NT>((g & 1) ? As0 : As1, (g & 1) ? Bs0 : Bs1, wm, wn, fr, fh, 0, fa0, fb0);
      if (g + 2 < G) issue(g + 2);
      __builtin_amdgcn_sched_barrier(0);
      if (KS == 2 || !skip_hi) dl_mfmas<T, MT, NT>(fa1, fb1, acc);
      __builtin_amdgcn_sched_barrier(0);
      ++g;
    };
    chunk(std::true_type{}, half_tail && nchunks == 1);
    for (int c = 1; c < nchunks; ++c) chunk(std::false_type{}, half_tail && c == nchunks - 1);
    // epilogue of the column step: complex SNR of 8 templates per lane per
    // row tile, running peaks
    const int64_t n0 = ws + (int64_t)(st0 + st) * BN;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int64_t col = n0 + wn * 32 * NT + nt * 32 + fr;
      const bool ok = col < we;
      const int rel = (int)(col - ws);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          const float re = acc[mt][nt][2 * p], im = acc[mt][nt][2 * p + 1];
          const float v = re * re + im * im;
          if (ok && v > best[mt][p].v) best[mt][p] = VN{v, rel};
          if (SNR && ok) {
            const int64_t i = (r0 + wm * 32 * MT + mt * 32 + 8 * (p >> 1) + 4 * fh + 2 * (p & 1)) >> 1;
            if (i < n_templates) {
              // written once and not read here: a non-temporal store
              typedef float fv2 __attribute__((ext_vector_type(2)));
              __builtin_nontemporal_store(fv2{re * inv_scale, im * inv_scale},
                                          (fv2 *)(jb.snr + (i * jb.snr_ld + (col - jb.snr_abs0)) * 2));
            }
          }
        }
      }
    }
  }

  // reduce the 32 columns of each half-wave, then the waves that share rows
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      VN bb = best[mt][p];
#pragma unroll
      for (int off = 1; off < 32; off <<= 1) {
        const float ov = __shfl_xor(bb.v, off);
        const int on = __shfl_xor(bb.n, off);
        if (better(ov, on, bb.v, bb.n)) bb = VN{ov, on};
      }
      if (fr == 0) red[wn][wm * 16 * MT + mt * 16 + 4 * (p >> 1) + 2 * fh + (p & 1)] = bb;
    }
  __syncthreads();
  for (int t = threadIdx.x; t < BM / 2; t += THREADS) {
    VN bb = red[0][t];
#pragma unroll
    for (int q = 1; q < WN; ++q)
      if (better(red[q][t].v, red[q][t].n, bb.v, bb.n)) bb = red[q][t];
    const int64_t i = r0 / 2 + t;
    if (i < n_templates) put_peak(jb, i, w, bb);
  }
}

// Phase and sub-sample refinement at each reported window peak: z_i at n* - 1,
// n*, n* + 1 recomputed as the dot products of mixing rows 2i, 2i+1 with those
// operand rows (FP32 accumulation; the operand holds one extra sample on each
// side of a chunk).  The refinement is the vertex of the parabola through the
// three |z| values (offset clipped to half a sample; none when the triple is
// not concave).  Peaks below `thr` get zeros (not reported).  The kernel first
// turns the mixing kernels' peak keys into |z| and the peak sample.
// One thread per (template, window) entry tests the threshold and writes the
// zeros; then the whole wave takes its entries above it two at a time: lane k
// reads 16-byte vector k of each of the 5 rows of both (all 10 reads in
// flight at once) and the 12 partial sums are reduced over the wave.  A pair
// is a round trip to memory and a wave takes its pairs one after another, so
// a table too small to fill the chip with waves of 64 entries gives each wave
// fewer (`per`, a power of two down to one pair): with every entry reported,
// 4514 entries of a BF16 bank 104 -> 8.4 us and 49152 of an FP32 one 112 ->
// 43 us.
template <typename T> struct Vec16 {
  T v[16 / sizeof(T)];
};

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

template <typename T>
__global__ __launch_bounds__(256) void k_peak_phase(const MixJob *__restrict__ jobs, int n_jobs, int64_t entries,
                                                    int per, float thr, float trig_thr,
                                                    int64_t *__restrict__ counts,
                                                    int32_t *__restrict__ xi_counters) {
  const int lane = threadIdx.x & 63;
  const int64_t e = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * per + lane;
  int job = 0;
  int64_t o = 0, row = 0, pn = 0;   // peak-table offset, template and peak sample of this lane's entry
  int64_t blk = -1;         // trigger-compaction block it counts in, if it is a trigger
  bool hit = false;
  // the signal-consistency launches, next in the stream, start from zero counters
  if (xi_counters && blockIdx.x == 0 && threadIdx.x < 2) xi_counters[threadIdx.x] = 0;
  if (lane < per && e < entries) {
    // job owning entry e: last job with e0 <= e
    int lo = 0, hi = n_jobs - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (jobs[mid].e0 <= e) lo = mid;
      else hi = mid - 1;
    }
    job = lo;
    const MixJob &jb = jobs[lo];
    const int64_t le = e - jb.e0;
    row = le / jb.nw;
    const int64_t w = jb.w0 + le - row * jb.nw;
    o = row * jb.ld_peak + (w - jb.w_base);
    // the mixing kernels leave the peak as a key (peak_key) in the sample's place
    const VN pk = peak_of_key(((const uint64_t *)jb.peak_n)[o]);
    const float snr = sqrtf(fmaxf(pk.v, 0.f)) * jb.inv_scale;
    pn = (w * jb.win_p) / jb.win_q + pk.n;
    jb.peak_snr[o] = snr;
    jb.peak_n[o] = pn;
    hit = snr >= thr && pk.v >= 0.f;   // (a window of NaNs only has no peak sample)
    if (snr >= trig_thr) blk = (jb.t0 + o) / kTrigPerBlock;
    if (!hit) {
      jb.peak_phase[o] = 0.f;
      jb.peak_dt[o] = 0.f;
      jb.peak_si[o] = 0.f;
    }
  }
  // triggers per compaction block: a wave's entries fall into few blocks
  uint64_t left = __ballot(blk >= 0);
  while (left) {
    const int s0 = __builtin_ctzll(left);
    const int64_t b0 = ((int64_t)__builtin_amdgcn_readlane((int)(blk >> 32), s0) << 32) |
                       (uint32_t)__builtin_amdgcn_readlane((int)blk, s0);
    const uint64_t same = __ballot(blk == b0);
    if (lane == s0) atomicAdd((unsigned long long *)(counts + b0), (unsigned long long)__popcll(same));
    left &= ~same;
  }
  constexpr int EPV = 16 / (int)sizeof(T);
  uint64_t m = __ballot(hit);
  while (m) {
    // up to two entries of the wave; the second repeats the first when there is none
    const int s0 = __builtin_ctzll(m);
    m &= m - 1;
    const int s1 = m ? __builtin_ctzll(m) : s0;
    if (m) m &= m - 1;
    const int src[2] = {s0, s1};
    float acc[2][6];
    int jx[2];
    int64_t ox[2];
    const uint4 *mc[2], *ms[2], *o0[2];
    int nv[2], pv[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      jx[t] = __builtin_amdgcn_readlane(job, src[t]);
      const MixJob &jb = jobs[jx[t]];
      const int64_t r = ((int64_t)__builtin_amdgcn_readlane((int)(row >> 32), src[t]) << 32) |
                        (uint32_t)__builtin_amdgcn_readlane((int)row, src[t]);
      ox[t] = ((int64_t)__builtin_amdgcn_readlane((int)(o >> 32), src[t]) << 32) |
              (uint32_t)__builtin_amdgcn_readlane((int)o, src[t]);
      const int64_t n = ((int64_t)__builtin_amdgcn_readlane((int)(pn >> 32), src[t]) << 32) |
                        (uint32_t)__builtin_amdgcn_readlane((int)pn, src[t]);
      // kcat and the row pitch kld are multiples of 32: whole 16-byte vectors
      nv[t] = jb.kcat / EPV;
      pv[t] = jb.kld / EPV;
      o0[t] = (const uint4 *)((const T *)jb.ocat + (n - 1 - jb.ocat_abs0) * (int64_t)jb.kld);
      mc[t] = (const uint4 *)((const T *)jb.mix + (2 * r) * (int64_t)jb.kld);
      ms[t] = mc[t] + pv[t];
#pragma unroll
      for (int q = 0; q < 6; ++q) acc[t][q] = 0.f;
    }
    for (int k0 = 0; k0 < max(nv[0], nv[1]); k0 += 64) {
      const int k = k0 + lane;
      Vec16<T> c[2], d[2], a[2][3];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const bool ok = k < nv[t];
        const int kk = ok ? k : 0;
        c[t] = __builtin_bit_cast(Vec16<T>, mc[t][kk]);
        d[t] = __builtin_bit_cast(Vec16<T>, ms[t][kk]);
#pragma unroll
        for (int q = 0; q < 3; ++q) a[t][q] = __builtin_bit_cast(Vec16<T>, o0[t][q * pv[t] + kk]);
        if (!ok) c[t] = d[t] = Vec16<T>{};
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
          for (int j = 0; j < EPV; ++j) {
            // explicit FMAs: the same arithmetic in both slots (the compiler
            // would otherwise pair some products into dot-product
            // instructions that round differently)
            const float ov = Op<T>::tof(a[t][q].v[j]);
            acc[t][q] = __builtin_fmaf(Op<T>::tof(c[t].v[j]), ov, acc[t][q]);
            acc[t][3 + q] = __builtin_fmaf(Op<T>::tof(d[t].v[j]), ov, acc[t][3 + q]);
          }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int q = 0; q < 6; ++q) acc[t][q] = wave_sum(acc[t][q]);
    if (lane == 0) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        if (t == 1 && s1 == s0) break;
        const MixJob &jb = jobs[jx[t]];
        const float *re = acc[t], *im = acc[t] + 3;
        float amp[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) amp[q] = sqrtf(re[q] * re[q] + im[q] * im[q]) * jb.inv_scale;
        const float curv = amp[0] - 2.f * amp[1] + amp[2];
        float dt = 0.f, v = amp[1];
        if (curv < 0.f) {
          dt = fminf(0.5f, fmaxf(-0.5f, (amp[0] - amp[2]) / (2.f * curv)));
          v = amp[1] - 0.25f * (amp[0] - amp[2]) * dt;
        }
        jb.peak_phase[ox[t]] = atan2f(im[1], re[1]);
        jb.peak_dt[ox[t]] = dt;
        jb.peak_si[ox[t]] = v;
        if (jb.peak_z) jb.peak_z[ox[t]] = make_float2(re[1] * jb.inv_scale, im[1] * jb.inv_scale);
      }
    }
  }
}

// Signal-consistency value at each trigger peak (Sec. II.A computes phase and
// xi^2 for every trigger):
//   xi2 = sum_k |z[n* + k] - z[n*] R[k]|^2 / sum_k (2 - 2 |R[k]|^2)
// over the lags k = -K..K with 0 <= n* + k < n_end.  z is recomputed at the
// lags as MFMA tiles Z = M_rows * Ocat^T over groups of 16 triggers (32
// mixing rows: cos and sin of 16 templates) and 32 samples; the tile's
// epilogue adds each lane's lags to its eight triggers' sums, and z[n*] comes
// from the phase kernel.  Triggers are listed per window and sorted by peak
// sample, so that a group's lags lie close together: the samples a group
// covers are about its spread of peaks plus 2K (a chunk's operand holds K
// extra samples on each side).
//
// Two forms.  16-bit operands with kcat <= 512 (and autocorrelation tables
// of fewer than 2^31 entries) run two launches:
// k_xi2_list (one workgroup per (job, window)) stores the sorted keys and
// appends one unit per 64 of them to a list, and k_xi2_tiles (persistent
// workgroups taking units from that list) keeps each wave's A fragments in
// registers for the whole unit and stages every operand tile once in LDS for
// its four waves, with coalesced direct-to-LDS loads.  Otherwise k_xi2 does
// both in one workgroup per (job, window), reading fragments straight from
// memory.

constexpr int kXiThreads = 256;
constexpr int kXiList = 1024;   // triggers listed per pass over a window's templates
constexpr int kXiGroup = 16;    // triggers per MFMA row tile

// (job, window) item `item` of the signal-consistency launches: the last job
// with x0 <= item.
__device__ __forceinline__ int find_xi_job(const MixJob *__restrict__ jobs, int n_jobs, int64_t item) {
  int lo = 0, hi = n_jobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].x0 <= item) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// One listing pass of window w (start ws) over templates [i0, F): the keys
// (n* - ws) << 32 | i of at most kXiList triggers in l_key, sorted by peak
// sample (template order among equal samples).  Returns how many; *i_next is
// the first template left for the next pass (F when none).  Every thread of
// the workgroup calls it.
__device__ int xi_list_pass(const MixJob &jb, int64_t w, int64_t ws, float thr, int i0, int64_t *l_key,
                            int *l_count, int *i_next_out) {
  const int F = jb.n_templates, lane = threadIdx.x & 63;
  if (threadIdx.x == 0) *l_count = 0;
  __syncthreads();
  int i_next = F;
  for (int ib = i0; ib < F; ib += kXiThreads) {
    const int i = ib + (int)threadIdx.x;
    const int64_t o = (int64_t)i * jb.ld_peak + (w - jb.w_base);
    const bool f = i < F && jb.peak_snr[o] >= thr;
    const uint64_t m = __ballot(f);
    int base = 0;
    if (lane == 0 && m) base = atomicAdd(l_count, (int)__popcll(m));
    base = __shfl(base, 0);
    if (f) {
      const int at = base + (int)__popcll(m & (lane ? (~0ull >> (64 - lane)) : 0ull));
      if (at < kXiList) l_key[at] = ((jb.peak_n[o] - ws) << 32) | (int64_t)i;
    }
    __syncthreads();
    const int cnt = *l_count;
    __syncthreads();
    if (cnt > kXiList) {   // full: this block's triggers wait for the next pass
      i_next = ib;
      break;
    }
  }
  int n_list = min(*l_count, kXiList);
  if (i_next < F) {
    // keep the triggers of templates below i_next (every one of them fits)
    __syncthreads();
    if (threadIdx.x == 0) {
      int k = 0;
      for (int t = 0; t < n_list; ++t)
        if ((int)(l_key[t] & 0xffffffff) < i_next) l_key[k++] = l_key[t];
      *l_count = k;
    }
    __syncthreads();
    n_list = *l_count;
  }
  // bitonic sort of the keys by peak sample (padding sorts last)
  int np2 = 1;
  while (np2 < n_list) np2 <<= 1;
  for (int t = n_list + (int)threadIdx.x; t < np2; t += kXiThreads) l_key[t] = INT64_MAX;
  __syncthreads();
  for (int size = 2; size <= np2; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int t = threadIdx.x; t < np2 / 2; t += kXiThreads) {
        const int a = 2 * stride * (t / stride) + (t % stride), b2 = a + stride;
        const bool up = (a & size) == 0;
        const int64_t x = l_key[a], y = l_key[b2];
        if ((x > y) == up) {
          l_key[a] = y;
          l_key[b2] = x;
        }
      }
      __syncthreads();
    }
  *i_next_out = i_next;
  return n_list;
}

template <typename T>
__global__ __launch_bounds__(kXiThreads) void k_xi2(const MixJob *__restrict__ jobs, int n_jobs, float thr) {
  typedef Op<T> O;
  __shared__ int64_t l_key[kXiList];   // (n* - window start) << 32 | template
  __shared__ int l_count;

  // job and window of this workgroup
  const int64_t item = blockIdx.x;
  const MixJob &jb = jobs[find_xi_job(jobs, n_jobs, item)];
  const int64_t wl = item - jb.x0;
  if (!jb.acorr || wl >= jb.nw) return;   // uniform over the workgroup
  const int64_t w = jb.w0 + wl;
  const int64_t ws = (w * jb.win_p) / jb.win_q;
  const int K = jb.acorr_half, kcat = jb.kcat, F = jb.n_templates;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const T *mix = (const T *)jb.mix;
  const T *ocat = (const T *)jb.ocat;
  const float2 *acorr = (const float2 *)jb.acorr;
  const float sc = jb.inv_scale;
  const int nks = kcat / O::KS;

  for (int i0 = 0; i0 < F;) {
    int i_next;
    const int n_list = xi_list_pass(jb, w, ws, thr, i0, l_key, &l_count, &i_next);

    // ---- groups of kXiGroup triggers, one wave each
    const int n_groups = (n_list + kXiGroup - 1) / kXiGroup;
    for (int g = wave; g < n_groups; g += kXiThreads / 64) {
      const int t0 = g * kXiGroup, nt = min(kXiGroup, n_list - t0);
      // A rows: lane row rr = lane % 32 is cos (even) or sin (odd) of trigger rr / 2
      const int tr = (lane & 31) >> 1;
      const int64_t ir = l_key[t0 + (tr < nt ? tr : 0)] & 0xffffffff;
      const T *arow = mix + (2 * ir + (lane & 1)) * (int64_t)jb.kld + (lane >> 5) * O::VEC;
      // the eight triggers of this lane's accumulator pairs: rows 8 (e/4) + 4 (lane/32) + e%4
      int64_t ns[8], ii[8];
      float2 zs[8];
      float num[8], den[8];
#pragma unroll
      for (int p = 0; p < 8; ++p) {
        const int tq = 4 * (p >> 1) + 2 * (lane >> 5) + (p & 1);
        const int64_t key = l_key[t0 + (tq < nt ? tq : 0)];
        ns[p] = tq < nt ? ws + (key >> 32) : INT64_MIN / 4;   // absent triggers reach no lag
        ii[p] = key & 0xffffffff;
        const float2 z = jb.peak_z[ii[p] * jb.ld_peak + (w - jb.w_base)];
        zs[p] = z;
        num[p] = 0.f;
        den[p] = 0.f;
      }
      // samples the group's lags reach, inside the data
      int64_t a0 = ws + (l_key[t0] >> 32) - K, a1 = ws + (l_key[t0 + nt - 1] >> 32) + K + 1;
      if (a0 < 0) a0 = 0;
      if (a1 > jb.n_end) a1 = jb.n_end;
      // blocks of U = 10 k-steps when that takes fewer blocks than U = 8 (30
      // k-steps: 3 instead of 4), else 8; more staging registers than 10 per
      // block would halve the occupancy
      auto tiles = [&](auto u_const) {
        constexpr int U = decltype(u_const)::value;
        for (int64_t s0 = a0; s0 < a1; s0 += 32) {
          const int64_t n = s0 + (lane & 31);
          const int64_t nb = n < a1 ? n : a1 - 1;
          const T *brow = ocat + (nb - jb.ocat_abs0) * (int64_t)jb.kld + (lane >> 5) * O::VEC;
          // two accumulators (even and odd k-steps) halve the MFMA dependency
          // chain.  Blocks of U k-steps issue all their reads before their MFMAs;
          // in the last block the k-steps past nks read k-step nks - 1 (in
          // range) and multiply a zero operand, so no k-step waits on its own
          // read alone and the block has no branches.
          f32x16 acc, acc2;
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[e] = acc2[e] = 0.f;
          for (int ks = 0; ks < nks; ks += U) {
            typename O::vec af[U], bf[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const int k = min(ks + u, nks - 1);
              af[u] = *(const typename O::vec *)(arow + k * O::KS);
              bf[u] = *(const typename O::vec *)(brow + k * O::KS);
              if (ks + u >= nks) bf[u] = typename O::vec{};
            }
            __builtin_amdgcn_sched_barrier(0);   // keep the block's reads ahead of its MFMAs
#pragma unroll
            for (int u = 0; u < U; u += 2) {
              acc = O::mfma(af[u], bf[u], acc);
              acc2 = O::mfma(af[u + 1], bf[u + 1], acc2);
            }
          }
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[e] += acc2[e];
#pragma unroll
          for (int p = 0; p < 8; ++p) {
            const int64_t lag = n - ns[p];
            if (n < a1 && lag >= -K && lag <= K) {
              const float2 r = acorr[ii[p] * (2 * K + 1) + K + lag];
              const float dr = acc[2 * p] * sc - (zs[p].x * r.x - zs[p].y * r.y);
              const float di = acc[2 * p + 1] * sc - (zs[p].x * r.y + zs[p].y * r.x);
              num[p] += dr * dr + di * di;
              den[p] += 2.f - 2.f * (r.x * r.x + r.y * r.y);
            }
          }
        }
      };
      if ((nks + 9) / 10 < (nks + 7) / 8) tiles(std::integral_constant<int, 10>{});
      else tiles(std::integral_constant<int, 8>{});
      // sum each trigger's terms over the 32 lanes (samples) of its half-wave
#pragma unroll
      for (int p = 0; p < 8; ++p)
        for (int off = 1; off < 32; off <<= 1) {
          num[p] += __shfl_xor(num[p], off);
          den[p] += __shfl_xor(den[p], off);
        }
      if ((lane & 31) == 0) {
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          const int tq = 4 * (p >> 1) + 2 * (lane >> 5) + (p & 1);
          if (tq < nt) jb.peak_xi[ii[p] * jb.ld_peak + (w - jb.w_base)] = den[p] > 0.f ? num[p] / den[p] : 0.f;
        }
      }
    }
    __syncthreads();
    i0 = i_next;
  }
}

// Listing launch of the two-launch form: keys of window w go to the job's
// listing slab at xi_key[(w - w_base) F + t], t = 0..count - 1 (one sorted
// run per listing pass), and units (item, 64 j, min(64, count - 64 j)) to
// units[counters[0]++ ...].  The phase kernel has zeroed the counters.
__global__ __launch_bounds__(kXiThreads) void k_xi2_list(const MixJob *__restrict__ jobs, int n_jobs, float thr,
                                                         XiUnit *__restrict__ units, int64_t cap,
                                                         int32_t *__restrict__ counters) {
  __shared__ int64_t l_key[kXiList];
  __shared__ int l_count, l_u0;
  const int64_t item = blockIdx.x;
  const MixJob &jb = jobs[find_xi_job(jobs, n_jobs, item)];
  const int64_t wl = item - jb.x0;
  if (!jb.acorr || wl >= jb.nw) return;   // uniform over the workgroup
  const int64_t w = jb.w0 + wl;
  const int64_t ws = (w * jb.win_p) / jb.win_q;
  const int F = jb.n_templates;
  int64_t *slab = jb.xi_key + (w - jb.w_base) * (int64_t)F;
  int count = 0;
  for (int i0 = 0; i0 < F;) {
    int i_next;
    const int n_list = xi_list_pass(jb, w, ws, thr, i0, l_key, &l_count, &i_next);
    for (int t = threadIdx.x; t < n_list; t += kXiThreads) slab[count + t] = l_key[t];
    count += n_list;
    __syncthreads();   // the next pass rewrites l_key
    i0 = i_next;
  }
  const int nu = (count + 63) / 64;
  if (nu == 0) return;
  if (threadIdx.x == 0) l_u0 = atomicAdd(&counters[0], nu);
  __syncthreads();
  for (int j = threadIdx.x; j < nu; j += kXiThreads) {
    const int64_t u = (int64_t)l_u0 + j;
    if (u < cap) units[u] = XiUnit{item, 64 * j, min(64, count - 64 * j)};
  }
}

// Staged operand tile: 32 rows (samples) of kcat 16-bit values, row pitch P =
// kcat / 8 + 1 16-byte chunks (odd, so 16 consecutive rows start on distinct
// banks): at most 33 loads of 64 chunks for kcat = 512.
constexpr int kXiTileBlocks = 33;
constexpr int kXiLoads = 9;   // loads per wave and tile: 4 waves x 9 >= kXiTileBlocks

// Tile launch of the two-launch form.  Workgroups take units from
// counters[1] until the list of counters[0] units is done.  Wave g of a unit
// owns its triggers 16 g .. 16 g + 15: the A fragments of every k-step stay in
// registers (NKS >= kcat / 16 k-steps; the ones past kcat are zeros) and its
// lag range [ga0, ga1) decides which tiles it multiplies.  The workgroup walks
// the union [ba0, ba1) of its waves' ranges in 32-sample tiles; each tile is
// loaded once into LDS, double-buffered.  Every wave issues exactly kXiLoads
// loads per tile (the ones past the tile land in a scratch block) and always
// issues the next tile (past the range: zeros), and the tile's
// autocorrelation reads go out before those loads: loads complete in issue
// order, so the epilogue then waits for its own reads only, not for the
// next tile.
template <typename T, int NKS>
__global__ __launch_bounds__(kXiThreads, 2) void k_xi2_tiles(const MixJob *__restrict__ jobs, int n_jobs,
                                                             const XiUnit *__restrict__ units, int64_t cap,
                                                             int32_t *__restrict__ counters) {
  static_assert(sizeof(T) == 2, "16-bit operands only");
  static_assert(NKS % 4 == 0 && NKS <= 32, "k-steps in blocks of 4, kcat <= 512");
  static_assert(4 * kXiLoads >= kXiTileBlocks, "whole tiles");
  typedef typename Op<T>::vec vec;
  __shared__ __attribute__((aligned(1024))) char Bt[2][kXiTileBlocks * 1024];
  __shared__ __attribute__((aligned(1024))) char Bx[1024];   // landing block of the loads past a tile
  __shared__ int64_t s_key[64];
  __shared__ float2 s_z[64];
  __shared__ int s_lo[64], s_ab[64];   // lag window start (relative to ws), autocorrelation row
  __shared__ int s_u;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 31, fh = lane >> 5;
  const int64_t n_units = min((int64_t)counters[0], cap);
  for (;;) {
    if (threadIdx.x == 0) s_u = atomicAdd(&counters[1], 1);
    __syncthreads();
    const int u = __builtin_amdgcn_readfirstlane(s_u);   // the same in every lane: keep it scalar
    if (u >= n_units) break;                              // uniform over the workgroup
    const XiUnit un = units[u];
    const MixJob &jb = jobs[find_xi_job(jobs, n_jobs, un.item)];
    const int64_t w = jb.w0 + (un.item - jb.x0);
    const int64_t ws = (w * jb.win_p) / jb.win_q;
    const int64_t pcol = w - jb.w_base;
    const int K = jb.acorr_half, kcat = jb.kcat, nks = kcat / 16, nt_u = un.n;
    if (threadIdx.x < 64) {
      int64_t key = -1;
      float2 z = make_float2(0.f, 0.f);
      int lo = INT_MIN / 2, ab = 0;   // a missing trigger reaches no lag
      if (lane < nt_u) {
        key = jb.xi_key[pcol * jb.n_templates + un.first + lane];
        z = jb.peak_z[(key & 0xffffffff) * jb.ld_peak + pcol];
        lo = (int)(key >> 32) - K;
        ab = (int)(key & 0xffffffff) * (2 * K + 1);
      }
      s_key[lane] = key;
      s_z[lane] = z;
      s_lo[lane] = lo;
      s_ab[lane] = ab;
    }
    __syncthreads();

    // peak samples (relative to ws): range of this wave's group, then of the unit
    const int nr_l = (int)(s_key[lane] >> 32);
    int mn = lane < nt_u ? nr_l : INT_MAX, mx = lane < nt_u ? nr_l : INT_MIN;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
      mn = min(mn, __shfl_xor(mn, off));
      mx = max(mx, __shfl_xor(mx, off));
    }
    const int gmn = __builtin_amdgcn_readfirstlane(__shfl(mn, 16 * wave));
    const int gmx = __builtin_amdgcn_readfirstlane(__shfl(mx, 16 * wave));
#pragma unroll
    for (int off = 16; off < 64; off <<= 1) {
      mn = min(mn, __shfl_xor(mn, off));
      mx = max(mx, __shfl_xor(mx, off));
    }
    mn = __builtin_amdgcn_readfirstlane(mn);
    mx = __builtin_amdgcn_readfirstlane(mx);
    const int64_t ba0 = max<int64_t>(0, ws + mn - K), ba1 = min<int64_t>(jb.n_end, ws + mx + K + 1);
    const bool has = 16 * wave < nt_u;
    const int64_t ga0 = has ? max<int64_t>(0, ws + gmn - K) : INT64_MAX;
    const int64_t ga1 = has ? min<int64_t>(jb.n_end, ws + gmx + K + 1) : INT64_MIN;

    // A fragments: lane row fr is cos (even) or sin (odd) of trigger 16 g + fr / 2
    // (a missing trigger repeats the unit's first; its rows are never used)
    vec af[NKS];
    {
      const int tr = 16 * wave + (fr >> 1);
      const int64_t i = s_key[tr < nt_u ? tr : 0] & 0xffffffff;
      const T *arow = (const T *)jb.mix + (2 * i + (lane & 1)) * (int64_t)jb.kld + fh * 8;
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        const vec v = *(const vec *)(arow + min(ks, nks - 1) * 16);
        af[ks] = ks < nks ? v : vec{};
      }
    }
    float num[8], den[8];
#pragma unroll
    for (int p = 0; p < 8; ++p) num[p] = den[p] = 0.f;

    // tile loads: this wave's load i fills block 4 i + wave of the tile, lane
    // chunk c = 64 (4 i + wave) + lane = row c / P, position c % P (the pad
    // position reads the row's first chunk, rows past 31 read row 31).  The
    // resource ends at the unit's last sample: rows past it load zeros, and
    // so do the blocks past the tile's nblk (into Bx past kXiTileBlocks).
    const int cpr = kcat / 8, P = cpr + 1, nblk = (32 * P + 63) / 64;
    // the resource starts at the unit's first operand row (its extent is the
    // unit's lag range, not the whole operand)
    const int rowbytes = jb.kld * 2;   // operand row pitch
    const __amdgpu_buffer_rsrc_t rb =
        make_rsrc((const T *)jb.ocat + (ba0 - jb.ocat_abs0) * (int64_t)jb.kld, (ba1 - ba0) * (int64_t)rowbytes);
    const int dr = 256 / P, dq = 256 - dr * P;
    const int base0 = 0;
    auto issue = [&](int j) {
      // the chunk positions are recomputed per tile (a few ALU operations per
      // load) rather than held in registers across the loop
      int c0 = wave * 64 + lane;
      asm volatile("" : "+v"(c0));
      int r = c0 / P, q = c0 - r * P;
      const int tb = base0 + 32 * j * rowbytes;
      char *buf = Bt[j & 1];
#pragma unroll
      for (int i = 0; i < kXiLoads; ++i) {
        const int blk = 4 * i + wave;
        const int vo = blk < nblk ? tb + min(r, 31) * rowbytes + (q < cpr ? q : 0) * 16 : 0x7ffffff0;
        char *dst = blk < kXiTileBlocks ? buf + blk * 1024 : Bx;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void *)dst, 16, vo, 0, 0, 0);
        q += dq;
        r += dr;
        if (q >= P) {
          q -= P;
          ++r;
        }
      }
    };
    const int ntl = (int)((ba1 - ba0 + 31) / 32);
    // a global (not generic) pointer: its reads count on the vector-memory
    // counter only, so the epilogue's wait leaves the next tile's loads in flight
    typedef float fv2 __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(1))) const fv2 gfv2;
    gfv2 *acorr = (gfv2 *)jb.acorr;
    const float sc = jb.inv_scale;
    const int nrel0 = (int)(ba0 - ws) + fr, nrel_end = (int)(ba1 - ws);
    issue(0);
    for (int j = 0; j < ntl; ++j) {
      __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wave's loads of tile j
      __syncthreads();                      // every wave's; tile j - 1's buffer is free
      // the lane's eight triggers (accumulator rows 8 (e/4) + 4 fh + e%4):
      // autocorrelation at this lane's lag of each (a lag outside the window
      // reads entry 0 and adds nothing)
      const int nrel = nrel0 + 32 * j;   // this lane's sample, relative to ws
      fv2 r[8];
      bool in[8];
#pragma unroll
      for (int p = 0; p < 8; ++p) {
        const int t = 16 * wave + 4 * (p >> 1) + 2 * fh + (p & 1);
        const int d = nrel - s_lo[t];
        in[p] = nrel < nrel_end && (unsigned)d <= (unsigned)(2 * K);
        r[p] = acorr[in[p] ? s_ab[t] + d : 0];
      }
      issue(j + 1);   // past the range: zeros into the free buffer
      const int64_t s0 = ba0 + 32 * (int64_t)j;
      if (s0 < ga1 && s0 + 32 > ga0) {   // uniform over the wave
        const char *bb = Bt[j & 1] + (fr * P + fh) * 16;
        f32x16 acc;
#pragma unroll
        for (int kb = 0; kb < NKS; kb += 4) {
          vec bf[4];
#pragma unroll
          for (int u2 = 0; u2 < 4; ++u2) bf[u2] = *(const vec *)(bb + (kb + u2) * 32);
          __builtin_amdgcn_sched_barrier(0);   // the block's reads ahead of its MFMAs
#pragma unroll
          for (int u2 = 0; u2 < 4; ++u2) acc = Op<T>::mfma(af[kb + u2], bf[u2], kb + u2 == 0 ? f32x16{} : acc);
        }
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          const float2 z = s_z[16 * wave + 4 * (p >> 1) + 2 * fh + (p & 1)];
          const float dre = acc[2 * p] * sc - (z.x * r[p].x - z.y * r[p].y);
          const float dim = acc[2 * p + 1] * sc - (z.x * r[p].y + z.y * r[p].x);
          if (in[p]) {
            num[p] += dre * dre + dim * dim;
            den[p] += 2.f - 2.f * (r[p].x * r[p].x + r[p].y * r[p].y);
          }
        }
      }
    }
    // sum each trigger's terms over the 32 lanes (samples) of its half-wave
#pragma unroll
    for (int p = 0; p < 8; ++p)
      for (int off = 1; off < 32; off <<= 1) {
        num[p] += __shfl_xor(num[p], off);
        den[p] += __shfl_xor(den[p], off);
      }
    if (fr == 0) {
#pragma unroll
      for (int p = 0; p < 8; ++p) {
        const int t = 16 * wave + 4 * (p >> 1) + 2 * fh + (p & 1);
        if (t < nt_u)
          jb.peak_xi[(s_key[t] & 0xffffffff) * jb.ld_peak + pcol] = den[p] > 0.f ? num[p] / den[p] : 0.f;
      }
    }
    // the zeros issued past the range have landed and every wave is done
    // with the unit's keys and tiles before the next unit reuses them
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();
  }
}

// ---------------------------------------------------------- trigger compaction
// Stream compaction over the flat (job, template, window) order of every peak
// table.  The phase kernel has counted the triggers of every block of
// kTrigPerBlock consecutive entries; a block's workgroup takes the sum of the
// counts before its own as its offset (each reads them all: up to
// kTrigInline blocks that is cheaper than a launch for the scan, 2 KB to 32
// KB from the L2 against 5 us) or, with more blocks, the offset that the scan
// launch has left, and rewrites its flagged entries from there, in
// kTrigPerBlock / 256 rounds of 256, so the cost follows the number of
// entries whatever the row shape.

constexpr int64_t kTrigInline = 4096;
constexpr int kTrigThreads = 256;

// Job owning flat entry e: the last job with elem0 <= e.
__device__ __forceinline__ int find_trig_job(const TrigJob *__restrict__ jobs, int n_jobs, int64_t e) {
  int lo = 0, hi = n_jobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].elem0 <= e) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ uint64_t lanes_below() {
  const int lane = (int)(threadIdx.x & 63);
  return lane ? (~0ull >> (64 - lane)) : 0ull;
}

// Exclusive prefix sum of counts[0..n) in place, total in *total; one block of
// 1024 threads, each taking 8 consecutive values per pass.
__global__ __launch_bounds__(1024) void k_trigger_scan(int64_t *counts, int64_t n, int64_t *total) {
  constexpr int V = 8, TPB = 1024;
  __shared__ int64_t wsum[TPB / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t carry = 0;
  for (int64_t base = 0; base < n; base += (int64_t)TPB * V) {
    const int64_t i0 = base + (int64_t)threadIdx.x * V;
    int64_t v[V];
    int64_t own = 0;
#pragma unroll
    for (int q = 0; q < V; ++q) {
      v[q] = i0 + q < n ? counts[i0 + q] : 0;
      own += v[q];
    }
    // inclusive scan of the per-thread sums across the wave, then across waves
    int64_t inc = own;
    for (int off = 1; off < 64; off <<= 1) {
      const int64_t u = __shfl_up(inc, off);
      if (lane >= off) inc += u;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int64_t before = carry, pass = 0;
    for (int q = 0; q < TPB / 64; ++q) {
      if (q < wave) before += wsum[q];
      pass += wsum[q];
    }
    int64_t run = before + inc - own;
#pragma unroll
    for (int q = 0; q < V; ++q) {
      if (i0 + q < n) counts[i0 + q] = run;
      run += v[q];
    }
    carry += pass;
    __syncthreads();
  }
  if (threadIdx.x == 0) *total = carry;
}

// SCANNED: counts holds the blocks' offsets; else their counts, and the last
// block writes the total (which may lie in host memory).
template <bool SCANNED>
__global__ __launch_bounds__(kTrigThreads) void k_trigger_write(const TrigJob *__restrict__ jobs, int n_jobs,
                                                                int64_t n_elems, float thr,
                                                                const int64_t *__restrict__ counts, int64_t cap,
                                                                lloid_trigger *__restrict__ out,
                                                                int64_t *__restrict__ total) {
  __shared__ int sh[kTrigThreads / 64];
  __shared__ int64_t sh_off[kTrigThreads / 64];
  const int wave = threadIdx.x >> 6;
  int64_t run = 0;
  if constexpr (SCANNED) {
    run = counts[blockIdx.x];
  } else {
    int64_t s = 0;
    for (int64_t q = threadIdx.x; q < (int64_t)blockIdx.x; q += kTrigThreads) s += counts[q];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if ((threadIdx.x & 63) == 0) sh_off[wave] = s;
    __syncthreads();
    for (int q = 0; q < kTrigThreads / 64; ++q) run += sh_off[q];
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = run + counts[blockIdx.x];
  }
  for (int k = 0; k < kTrigPerBlock / kTrigThreads; ++k) {
    const int64_t e = (int64_t)blockIdx.x * kTrigPerBlock + k * kTrigThreads + threadIdx.x;
    int j = 0;
    bool f = false;
    if (e < n_elems) {
      j = find_trig_job(jobs, n_jobs, e);
      f = jobs[j].snr[e - jobs[j].elem0] >= thr;
    }
    const uint64_t m = __ballot(f);
    if ((threadIdx.x & 63) == 0) sh[wave] = __popcll(m);
    __syncthreads();
    int64_t pos = run + __popcll(m & lanes_below());
    int blk = 0;
    for (int q = 0; q < kTrigThreads / 64; ++q) {
      if (q < wave) pos += sh[q];
      blk += sh[q];
    }
    if (f && pos < cap) {
      const TrigJob &jb = jobs[j];
      const int64_t o = e - jb.elem0;   // template o / nw, window o % nw of this table
      lloid_trigger t;
      t.bank = jb.bank_id;
      t.detector = jb.detector;
      t.template_id = (int32_t)(o / jb.nw);
      t.xi2 = jb.xi ? jb.xi[o] : 0.f;
      t.window = jb.w_base + o % jb.nw;
      t.sample = jb.peak_n[o];
      t.snr = jb.snr[o];
      t.phase = jb.phase[o];
      t.snr_interp = jb.si[o];
      t.dt = jb.dt[o];
      out[pos] = t;
    }
    run += blk;
    __syncthreads();
  }
}

// ---------------------------------------------------------- conditioning
// PSD, whitening and gating before the filter (Sec. II.A).  A segment of L
// samples (hop L/2, periodic Hann window) is transformed by L/8 threads with
// eight points each in registers: radix-2 Stockham stages taken three at a
// time, one LDS exchange per three stages (three exchanges per 4096-point
// transform; a barrier and a round trip per radix-2 stage, with the
// twiddles computed in place, took 59 us for the periodograms and 131 us for
// the whitening of 2^21 samples).  Twiddles and the window come from tables
// of the context.  The last stages leave point j + b L/8 in register b of
// thread j, the layout the input has, so whitening goes from the forward to
// the inverse transform without an exchange.  Every butterfly is the radix-2
// one (one product rounded, then a fused multiply-add), whatever the fusing.

// tw[ns + k] = (cos, sin)(pi k / ns), k < ns, for the radix-2 stage that
// combines transforms of ns points (ns = 1, 2, .. 2048): a stage's twiddles are
// contiguous in k, so a wave's read is a few lines (one half-turn table read
// with a stride per stage touched a line per lane).  win[n] = sin(pi n / 4096),
// n < 4096: shorter segments take every (4096 / L)-th entry.
constexpr int kFftMax = kCondMaxLen;

__global__ void k_fft_tables(float2 *__restrict__ tw, float *__restrict__ win) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i > 0 && i < kFftMax) {
    const int ns = 1 << (31 - __clz(i));
    float sn, cs;
    sincospif((float)(i - ns) / (float)ns, &sn, &cs);
    tw[i] = make_float2(cs, sn);
  }
  if (i < kFftMax) win[i] = sinpif((float)i / (float)kFftMax);
}

// (a, b) -> (a + w b, a - w b), w = cos + i SIGN sin of table entry t
template <int SIGN> __device__ __forceinline__ void fft_bfly(float2 &a, float2 &b, float2 t) {
  // the window or gain product that made a point is rounded before it is
  // added here: only the fused multiply-adds written out
#pragma clang fp contract(off)
  const float cs = t.x, sn = SIGN < 0 ? -t.y : t.y;
  const float tx = __builtin_fmaf(b.x, cs, -(b.y * sn)), ty = __builtin_fmaf(b.y, cs, b.x * sn);
  const float2 a0 = a;
  a = make_float2(a0.x + tx, a0.y + ty);
  b = make_float2(a0.x - tx, a0.y - ty);
}

// LDS place of point i: a pad every 8 points keeps the strided exchange
// writes off each other's banks
__device__ __forceinline__ int fft_place(int i) { return i + (i >> 3); }

// In-register transform of the segment's points v[c] = x[j + c L/8]; `buf` is
// the segment's exchange buffer of L 9/8 values.  Every thread of the
// workgroup calls it.
template <int LG, int SIGN>
__device__ __forceinline__ void fft_regs(float2 (&v)[8], float2 *buf, const float2 *__restrict__ tw, int j) {
  constexpr int NT = (1 << LG) / 8;
  constexpr int FULL = LG / 3, REM = LG % 3;
#pragma unroll
  for (int p = 0; p < FULL; ++p) {
    const int st = 3 * p, ns = 1 << st;
    const int k = j & (ns - 1), m = j >> st;
    // stage st pairs points c and c + 4, st + 1 points c and c + 2 of those, st + 2 neighbours;
    // v[c] then holds output (c bit 2, bit 1, bit 0) -> bits 0, 1, 2 of the output number
    const float2 t0 = tw[ns + k];
#pragma unroll
    for (int c = 0; c < 4; ++c) fft_bfly<SIGN>(v[c], v[c + 4], t0);
#pragma unroll
    for (int b0 = 0; b0 < 2; ++b0) {
      const float2 t1 = tw[2 * ns + b0 * ns + k];
      fft_bfly<SIGN>(v[4 * b0], v[4 * b0 + 2], t1);
      fft_bfly<SIGN>(v[4 * b0 + 1], v[4 * b0 + 3], t1);
    }
#pragma unroll
    for (int b0 = 0; b0 < 2; ++b0)
#pragma unroll
      for (int b1 = 0; b1 < 2; ++b1)
        fft_bfly<SIGN>(v[4 * b0 + 2 * b1], v[4 * b0 + 2 * b1 + 1], tw[4 * ns + (b0 + 2 * b1) * ns + k]);
    float2 o[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) o[b] = v[4 * (b & 1) + 2 * ((b >> 1) & 1) + (b >> 2)];
    if (p == FULL - 1 && REM == 0) {
#pragma unroll
      for (int b = 0; b < 8; ++b) v[b] = o[b];   // m = 0: output b sits at j + b L/8
    } else {
      if (p > 0) __syncthreads();                // the previous exchange has been read
#pragma unroll
      for (int b = 0; b < 8; ++b) buf[fft_place((m << (st + 3)) + (b << st) + k)] = o[b];
      __syncthreads();
#pragma unroll
      for (int c = 0; c < 8; ++c) v[c] = buf[fft_place(j + c * NT)];
    }
  }
  if constexpr (REM == 1) {
    // last stage: points j + c L/8 and the ones half a segment on, outputs in place
#pragma unroll
    for (int c = 0; c < 4; ++c) fft_bfly<SIGN>(v[c], v[c + 4], tw[4 * NT + j + c * NT]);
  }
  if constexpr (REM == 2) {
    // last two stages (ns = L/4, L/2): point c = 4 c2 + 2 m + c0 of thread j
    float2 o[8];
#pragma unroll
    for (int c0 = 0; c0 < 2; ++c0) {
      const float2 t = tw[2 * NT + j + c0 * NT];
      fft_bfly<SIGN>(v[c0], v[c0 + 4], t);           // m = 0: outputs b0 = 0, 1
      fft_bfly<SIGN>(v[c0 + 2], v[c0 + 6], t);       // m = 1
#pragma unroll
      for (int b0 = 0; b0 < 2; ++b0) {
        float2 x = v[c0 + 4 * b0], y = v[c0 + 2 + 4 * b0];
        fft_bfly<SIGN>(x, y, tw[4 * NT + j + (2 * b0 + c0) * NT]);
        o[2 * b0 + c0] = x;
        o[4 + 2 * b0 + c0] = y;
      }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = o[c];
  }
}

// Segments m = seg0 + 0 .. nseg - 1 cover samples [m L/2, m L/2 + L) of the
// strain (zero outside [0, T); converted to FP32 here, a sample that is not
// finite in FP32 counts as zero and is flagged by the whitening pass, whose
// segments cover every sample).  WHITEN = false: |X[f]|^2 for f <= L/2 into
// parts; true: X scaled by gain[min(f, L - f)], inverse transform, real part
// / L into y.  Workgroups of max(256, L/8) threads: 4096-point segments one
// each (36 KB of LDS, four workgroups per CU: every segment of 2^21 samples
// in flight at once), shorter ones several.
template <int LG> struct CondShape {
  static constexpr int L = 1 << LG, NT = L / 8;
  static constexpr int THREADS = NT > 256 ? NT : 256, SEGS = THREADS / NT;
};

template <int LG, bool WHITEN, typename TI>
__global__ __launch_bounds__(CondShape<LG>::THREADS) void k_cond_segment(
    const TI *__restrict__ x, int64_t T, int64_t seg0, int64_t nseg, const float2 *__restrict__ tw,
    const float *__restrict__ win, const float *__restrict__ gain, float *__restrict__ parts, float *__restrict__ y,
    int *__restrict__ bad, uint64_t *__restrict__ summary, int64_t n_summary) {
  typedef CondShape<LG> S;
  constexpr int L = S::L, NT = S::NT;
  __shared__ float2 buf[S::SEGS * (L + L / 8)];
  const int sg = threadIdx.x / NT, j = threadIdx.x % NT;
  const int64_t s = (int64_t)blockIdx.x * S::SEGS + sg;
  const bool live = s < nseg;
  const int64_t lo = (seg0 + s) * (L / 2);
  float2 v[8];
  bool finite = true;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int n = j + c * NT;
    const int64_t t = lo + n;
    float u = (live && t >= 0 && t < T) ? (float)x[t] : 0.f;
    if (!isfinite(u)) {
      finite = false;
      u = 0.f;
    }
    const float h = win[n * (kFftMax / L)];
    v[c] = make_float2(u * h * h, 0.f);
  }
  if (WHITEN && !finite) atomicOr(bad, 1);
  // the loud samples' summary bits, which the next launch sets (its T / 4032
  // words at most: L/8 threads for every L/2 samples are here)
  if constexpr (WHITEN) {
    const int64_t t = (int64_t)blockIdx.x * S::THREADS + threadIdx.x;
    if (t < n_summary) summary[t] = 0;
  }
  float2 *seg = buf + sg * (L + L / 8);
  fft_regs<LG, -1>(v, seg, tw, j);
  if constexpr (!WHITEN) {
    if (!live) return;
    float *out = parts + s * (L / 2 + 1);
#pragma unroll
    for (int b = 0; b < 4; ++b) out[j + b * NT] = __builtin_fmaf(v[b].x, v[b].x, v[b].y * v[b].y);
    if (j == 0) out[L / 2] = __builtin_fmaf(v[4].x, v[4].x, v[4].y * v[4].y);
  } else {
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const int f = j + b * NT;
      const float g = gain[f <= L / 2 ? f : L - f];
      v[b] = make_float2(v[b].x * g, v[b].y * g);
    }
    __syncthreads();   // the forward transform's last exchange has been read
    fft_regs<LG, 1>(v, seg, tw, j);
    if (!live) return;
    const float inv = 1.f / (float)L;
#pragma unroll
    for (int b = 0; b < 8; ++b) y[s * L + j + b * NT] = v[b].x * inv;
  }
}

__device__ __forceinline__ float psd_gain(float s, float f0) { return s > 0.f ? 1.f / sqrtf(s * f0 * 0.5f) : 0.f; }

// Per bin f <= L/2: the mean periodogram, c_f / (nseg f0 sum w^2) times the
// sum over segments (sum w^2 = 3 L / 8 for the periodic Hann window), and the
// whitening gain.  The sum over segments is compensated (Kahan): in FP32 its
// error stays at a few units of rounding whatever the number of segments.
// The sum is one dependent chain of four additions per segment, 64 bins to a
// wave, so the reads have to run ahead of it: four waves read the next
// 4 kPsdU segments into registers while the first adds the current ones from
// LDS.  1023 segments of 2049 bins: 255 us with a read per addition waited for
// in turn, 25 us with one wave reading 32 segments ahead, 19 us like this.
constexpr int kPsdU = 32;

__global__ __launch_bounds__(256) void k_psd_mean(const float *__restrict__ parts, int64_t nseg, int L, float f0,
                                                  float *__restrict__ psd, float *__restrict__ gain) {
  constexpr int U = kPsdU, TILE = 4 * U;
  __shared__ float tile[2][TILE][64];
  const int nf = L / 2 + 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int f = blockIdx.x * 64 + lane;
  const int fl = f < nf ? f : nf - 1;
  float r[U];
  // this wave's U segments of tile t (past the last segment: the last again, not added)
  auto read = [&](int64_t t) __attribute__((always_inline)) {
    const int64_t m0 = t * TILE + wave * U;
    const float *row = parts + min<int64_t>(m0, nseg - 1) * nf;
    const int more = (int)min<int64_t>(U, nseg - 1 - m0);   // steps that stay inside
#pragma unroll
    for (int u = 0; u < U; ++u) {
      r[u] = row[fl];
      row += u < more ? nf : 0;
    }
  };
  float acc = 0.f, comp = 0.f;
  const int64_t nt = (nseg + TILE - 1) / TILE;
  read(0);
  for (int64_t t = 0; t < nt; ++t) {
    float(*tl)[64] = tile[t & 1];
#pragma unroll
    for (int u = 0; u < U; ++u) tl[wave * U + u][lane] = r[u];
    __syncthreads();   // tile t is whole; tile t - 1 has been added (its buffer is next)
    if (t + 1 < nt) read(t + 1);
    if (wave == 0) {
      const int n = (int)min<int64_t>(TILE, nseg - t * TILE);
#pragma unroll 16
      for (int u = 0; u < n; ++u) {
        const float y = tl[u][lane] - comp;
        const float s = acc + y;
        comp = (s - acc) - y;
        acc = s;
      }
    }
  }
  if (wave != 0 || f >= nf) return;
  const float c = (f == 0 || f == L / 2) ? 1.f : 2.f;
  const float s = c * acc / ((float)nseg * f0 * (0.375f * (float)L));
  psd[f] = s;
  gain[f] = psd_gain(s, f0);
}

__global__ void k_psd_gain(const float *__restrict__ psd, int nf, float f0, float *__restrict__ gain) {
  const int f = blockIdx.x * blockDim.x + threadIdx.x;
  if (f < nf) gain[f] = psd_gain(psd[f], f0);
}

// out[n] = the two segments' outputs over sample n (segment m starts at m h,
// h = L/2 = 2^lgh; y holds segments seg0, seg0 + 1, ...).  loud: NULL, or one
// bit per sample, set where |out[n]| > thr, and their cleared summary bits.
constexpr int kOverlapPer = 4;   // samples per thread, 256 apart

__global__ __launch_bounds__(256) void k_overlap_add(const float *__restrict__ y, int64_t T, int lgh, int64_t seg0,
                                                     float thr, float *__restrict__ out,
                                                     uint64_t *__restrict__ loud) {
  const int64_t b0 = (int64_t)blockIdx.x * (256 * kOverlapPer) + threadIdx.x;
#pragma unroll
  for (int q = 0; q < kOverlapPer; ++q) {
    const int64_t n = b0 + 256 * q;
    bool l = false;
    if (n < T) {
      const int64_t mb = n >> lgh, ma = mb - 1;
      const float v = y[((ma - seg0) << (lgh + 1)) + (n - (ma << lgh))] +
                      y[((mb - seg0) << (lgh + 1)) + (n - (mb << lgh))];
      out[n] = v;
      l = fabsf(v) > thr;
    }
    if (loud) {
      const uint64_t m = __ballot(l);
      if ((threadIdx.x & 63) == 0 && n < T) {
        loud[n >> 6] = m;
        if (m)
          loud_mark(loud, T, n >> 6, [](uint64_t *p, uint64_t bit) {
            return (uint64_t)atomicOr((unsigned long long *)p, (unsigned long long)bit);
          });
      }
    }
  }
}

// Zeroes every sample within half_width of a loud one and counts them.  A
// workgroup first asks for any loud sample in its reach (its own samples and
// half_width on each side): transients are rare, so nearly all leave there.
// Latency decides: a reach of up to kGateWords words is read in one round, a word
// per thread; a longer one, and a sample's own question, take at most two words
// of each level, whatever the half width.  2^21 samples, half width 512: 4.8 us
// (8 with the second question alone); a call of 2^24 samples with a half width
// of 10^6: 436 us, with one loud sample 791, where reading every word in reach
// took 835 us and 16.2 ms.
constexpr int kGateSpan = 512;    // samples per workgroup
constexpr int kGateWords = 256;   // half widths up to 7900 samples

__global__ __launch_bounds__(256) void k_gate(const uint64_t *__restrict__ loud, int64_t T, int64_t half_width,
                                              float *__restrict__ out, unsigned long long *__restrict__ count) {
  const int64_t n0 = (int64_t)blockIdx.x * kGateSpan;
  const int64_t a0 = max<int64_t>(0, n0 - half_width), e0 = min<int64_t>(T - 1, n0 + kGateSpan - 1 + half_width);
  const int64_t w = (a0 >> 6) + threadIdx.x;
  if ((e0 >> 6) - (a0 >> 6) < kGateWords) {
    if (!__syncthreads_or(w <= (e0 >> 6) && loud[w])) return;
  } else if (!loud_any(loud, T, a0, e0)) {
    return;
  }
  bool g[kGateSpan / 256];
#pragma unroll
  for (int q = 0; q < kGateSpan / 256; ++q) {
    const int64_t n = n0 + q * 256 + threadIdx.x;
    g[q] = n < T && loud_any(loud, T, max<int64_t>(0, n - half_width), min<int64_t>(T - 1, n + half_width));
  }
#pragma unroll
  for (int q = 0; q < kGateSpan / 256; ++q) {
    if (g[q]) out[n0 + q * 256 + threadIdx.x] = 0.f;
    const uint64_t m = __ballot(g[q]);
    if ((threadIdx.x & 63) == 0 && m) atomicAdd(count, (unsigned long long)__popcll(m));
  }
}

// ---------------------------------------------------------- coincidence
// Pairs of triggers of two detectors with the same (bank, template) whose
// peak samples differ by at most max_dt (Sec. II.A, the coincidence
// generator).  Both lists are sorted by (bank, template, sample), so the
// partners of a[i] are one contiguous run of b, found by binary search; one
// thread per trigger of a counts its run, and the same threads write their pairs
// (a-major order) at the counts before theirs: the blocks' ones added up (or
// scanned, beyond kTrigInline blocks), their own block's scanned in place.  Per
// block, not per trigger, and without a launch for it: 2 x 126 thousand triggers
// 126 -> 26 us, of which the scan of one count per trigger in one workgroup
// took 98.  Both launches are bound by the 17 dependent reads of the search.

__device__ __forceinline__ bool key_before(const lloid_trigger &x, int32_t bank, int32_t tmpl, int64_t sample) {
  if (x.bank != bank) return x.bank < bank;
  if (x.template_id != tmpl) return x.template_id < tmpl;
  return x.sample < sample;
}

__device__ __forceinline__ bool out_of_order(const lloid_trigger &x, const lloid_trigger &y) {
  return key_before(y, x.bank, x.template_id, x.sample);
}

// first j with b[j] not before (bank, tmpl, sample - max_dt)
__device__ __forceinline__ int64_t coinc_first(const lloid_trigger *__restrict__ b, int64_t nb,
                                               const lloid_trigger &t, int64_t max_dt) {
  int64_t lo = 0, hi = nb;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (key_before(b[mid], t.bank, t.template_id, t.sample - max_dt)) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ bool coinc_partner(const lloid_trigger &x, const lloid_trigger &t, int64_t max_dt) {
  return x.bank == t.bank && x.template_id == t.template_id && x.sample <= t.sample + max_dt;
}

static_assert(kCoincThreads % 64 == 0, "whole waves");

__global__ __launch_bounds__(kCoincThreads) void k_coinc_count(const lloid_trigger *__restrict__ a, int64_t na,
                                                               const lloid_trigger *__restrict__ b, int64_t nb,
                                                               int64_t max_dt, int64_t *__restrict__ counts,
                                                               int *__restrict__ bad, uint8_t *__restrict__ bg_b) {
  __shared__ int64_t sh[kCoincThreads / 64];
  const int64_t i = (int64_t)blockIdx.x * kCoincThreads + threadIdx.x;
  bool unsorted = false;
  if (i < nb) {
    if (bg_b) bg_b[i] = 1;
    unsorted = i + 1 < nb && out_of_order(b[i], b[i + 1]);
  }
  int64_t c = 0;
  if (i < na) {
    const lloid_trigger t = a[i];
    unsorted = unsorted || (i + 1 < na && out_of_order(t, a[i + 1]));
    for (int64_t j = coinc_first(b, nb, t, max_dt); j < nb && coinc_partner(b[j], t, max_dt); ++j) ++c;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = c;
  const int any = __syncthreads_or(unsorted);
  if (threadIdx.x == 0) {
    int64_t sum = 0;
    for (int q = 0; q < kCoincThreads / 64; ++q) sum += sh[q];
    counts[blockIdx.x] = sum;
    bad[blockIdx.x] = any;
  }
}

// SCANNED: counts holds the blocks' offsets; else their counts, and the last
// block writes the total.  The last block also gathers the blocks' flags.
// res: the result words, in host memory.
template <bool SCANNED>
__global__ __launch_bounds__(kCoincThreads) void k_coinc_write(const lloid_trigger *__restrict__ a, int64_t na,
                                                               const lloid_trigger *__restrict__ b, int64_t nb,
                                                               int64_t max_dt, const int64_t *__restrict__ counts,
                                                               const int *__restrict__ bad, ResultWords *res,
                                                               int64_t cap, lloid_coinc *__restrict__ out,
                                                               uint8_t *__restrict__ bg_a, uint8_t *__restrict__ bg_b) {
  __shared__ int64_t sh[kCoincThreads / 64], sh_off[kCoincThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t m = 0;
  if constexpr (SCANNED) {
    m = counts[blockIdx.x];
  } else {
    int64_t s = 0;
    for (int64_t q = threadIdx.x; q < (int64_t)blockIdx.x; q += kCoincThreads) s += counts[q];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) sh_off[wave] = s;
    __syncthreads();
    for (int q = 0; q < kCoincThreads / 64; ++q) m += sh_off[q];
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) res->total = m + counts[blockIdx.x];
  }
  if (blockIdx.x == gridDim.x - 1) {
    bool f = false;
    for (int64_t q = threadIdx.x; q < (int64_t)gridDim.x; q += kCoincThreads) f = f || bad[q];
    const int any = __syncthreads_or(f);
    if (threadIdx.x == 0) res->bad = any;
  }
  const int64_t i = (int64_t)blockIdx.x * kCoincThreads + threadIdx.x;
  lloid_trigger t = {};
  int64_t j0 = 0, c = 0;
  if (i < na) {
    t = a[i];
    j0 = coinc_first(b, nb, t, max_dt);
    while (j0 + c < nb && coinc_partner(b[j0 + c], t, max_dt)) ++c;
    if (bg_a) bg_a[i] = c ? 0 : 1;
  }
  int64_t inc = c;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int64_t u = __shfl_up(inc, off);
    if (lane >= off) inc += u;
  }
  if (lane == 63) sh[wave] = inc;
  __syncthreads();
  for (int q = 0; q < wave; ++q) m += sh[q];
  m += inc - c;
  for (int64_t k = 0; k < c; ++k, ++m) {
    const int64_t j = j0 + k;
    const lloid_trigger u = b[j];
    if (bg_b) bg_b[j] = 0;
    if (m < cap) {
      lloid_coinc p;
      p.a = i;
      p.b = j;
      p.bank = t.bank;
      p.template_id = t.template_id;
      p.snr_net = sqrtf(t.snr * t.snr + u.snr * u.snr);
      p.dt = (float)(u.sample - t.sample) + (u.dt - t.dt);
      out[m] = p;
    }
  }
}

// ---------------------------------------------------------- tuning input
// Counter-based hash (the 32-bit finaliser of MurmurHash3 applied to the
// sample index and seed) mapped to a uniform value of unit variance.
__global__ void k_noise(float *__restrict__ x, int64_t n, uint32_t seed) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint32_t h = (uint32_t)i ^ (uint32_t)(i >> 32) * 0x9e3779b9u ^ seed;
  h ^= h >> 16;
  h *= 0x85ebca6bu;
  h ^= h >> 13;
  h *= 0xc2b2ae35u;
  h ^= h >> 16;
  x[i] = ((float)h * (1.f / 4294967296.f) - 0.5f) * 3.4641016f;
}

// ------------------------------------------------------------ launchers

static inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

hipError_t launch_ingest(const IngestArgs &a, lloid_dtype dt, hipStream_t s) {
  const unsigned tb = blocks_for(a.tab_vecs, 256), zb = blocks_for(a.zero_n, 256);
  const unsigned blocks = tb + zb + blocks_for(std::max<int64_t>(a.dst_len, 0), 256);
  if (!blocks) return hipSuccess;
  if (dt == LLOID_F64) k_ingest<double><<<blocks, 256, 0, s>>>(a, (int)tb, (int)zb);
  else k_ingest<float><<<blocks, 256, 0, s>>>(a, (int)tb, (int)zb);
  return hipGetLastError();
}

hipError_t launch_noise(float *x, int64_t n, uint32_t seed, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_noise<<<blocks_for(n, 256), 256, 0, s>>>(x, n, seed);
  return hipGetLastError();
}

hipError_t launch_decimate(DecimArgs a, hipStream_t s) {
  const int K = a.n_levels;
  if (K < 1 || K > kDecimGroup) return hipErrorInvalidValue;
  // the deepest level's samples over every level's wanted range
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  for (int k = 1; k <= K; ++k) {
    const DecimLevel &lv = a.level[k - 1];
    if (lv.hi <= lv.lo) continue;
    lo = std::min(lo, lv.lo >> (K - k));
    hi = std::max(hi, ((lv.hi - 1) >> (K - k)) + 1);
  }
  if (hi <= lo) return hipSuccess;
  // runs of 4096 finer-level samples, or of 1024 (four times as many halos) where
  // the long ones would leave CUs without a workgroup
  a.span = kDecimSpan >> K;
  if (hi - lo <= 256 * (int64_t)a.span) a.span = (kDecimSpan / 4) >> K;
  a.tile0 = floor_div(lo, a.span);
  k_decimate<<<(unsigned)(ceil_div(hi, a.span) - a.tile0), 256, 0, s>>>(a);
  return hipGetLastError();
}

template <typename T, int MT, int NT, int NW, int BK, bool HR = false, bool NARROW = false>
static hipError_t fir_v(const FirJob *jobs, int n_jobs, int64_t n_items, hipStream_t s) {
  k_fir<T, MT, NT, NW, BK, HR, NARROW><<<(unsigned)n_items, 64 * NW, 0, s>>>(jobs, n_jobs);
  return hipGetLastError();
}

template <typename T>
static hipError_t fir_t(int variant, const FirJob *jobs, int n_jobs, int64_t n_items, hipStream_t s) {
  switch (variant) {
    case 1: return fir_v<T, kFirMT, kFirNT, kFirWaves, kBK>(jobs, n_jobs, n_items, s);
    case 3:
    case 4:
      // 16-bit operands: the Hankel fragment window with basis chunks of 128
      // or 256 taps (a barrier per 8 or 16 k-steps instead of 4)
      if constexpr (sizeof(T) == 2) {
        if (variant == 3) return fir_v<T, 2, 4, kFirWaves, 4 * kBK, true>(jobs, n_jobs, n_items, s);
        return fir_v<T, 2, 4, kFirWaves, 8 * kBK, true>(jobs, n_jobs, n_items, s);
      } else {
        return fir_v<T, kFirMT, kFirNT, kFirWaves, kBK>(jobs, n_jobs, n_items, s);
      }
    case 5:
      // 16-bit operands: K chunks of 64 (twice the MFMAs per barrier)
      if constexpr (sizeof(T) == 2) return fir_v<T, kFirMT, kFirNT, kFirWaves, 2 * kBK>(jobs, n_jobs, n_items, s);
      else return fir_v<T, kFirMT, kFirNT, kFirWaves, kBK>(jobs, n_jobs, n_items, s);
    case 2:
      // 16-bit operands: 64 x 1024 tiles with the Hankel fragment window
      if constexpr (sizeof(T) == 2) return fir_v<T, 2, 4, kFirWaves, 2 * kBK, true>(jobs, n_jobs, n_items, s);
      else return fir_v<T, kFirMT, kFirNT, kFirWaves, kBK>(jobs, n_jobs, n_items, s);
    default:
      // 16-bit operands: the Hankel fragment window in four-wave 64 x 512
      // tiles, two workgroups per CU (one's strain-window fill and stores run
      // while the other's MFMAs do), basis chunks of 128 taps
      if constexpr (sizeof(T) == 2) return fir_v<T, 2, 4, 4, 4 * kBK, true, true>(jobs, n_jobs, n_items, s);
      else return fir_v<T, kFirMT, kFirNT, kFirWaves, kBK, false, true>(jobs, n_jobs, n_items, s);
  }
}

void fir_tile_shape(lloid_dtype t, int variant, int *bm, int *bn) {
  *bm = 32 * kFirMT;
  *bn = kFirWaves * 32 * kFirNT;
  if ((variant == 2 || variant == 3 || variant == 4) && t != LLOID_F32) *bm = 32 * 2, *bn = kFirWaves * 32 * 4;
  if (variant == 0 && t != LLOID_F32) *bm = 32 * 2, *bn = 4 * 32 * 4;
}

void fir_narrow_shape(int variant, int *bm, int *bn) {
  *bm = variant == 0 ? kFirNarrowBM : 0;
  *bn = variant == 0 ? kFirNarrowBN : 0;
}

void mix_tile_shape(lloid_dtype, int variant, int *bm, int *bn) {
  switch (variant) {
    case 1: *bm = 32 * 4 * 2, *bn = 32 * 2 * 2; break;
    case 2: *bm = 32 * 2 * 4, *bn = 32 * 2 * 2; break;
    case 3: *bm = 32 * kMixMT * kMixWM, *bn = 32 * kMixNT * kMixWN; break;
    default: *bm = 32 * kMixMT * kMixWM, *bn = 32 * kMixNT * kMixWN; break;
  }
}

hipError_t launch_fir_jobs(lloid_dtype t, int variant, const FirJob *jobs, int n_jobs, int64_t n_items,
                           hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  switch (t) {
    case LLOID_F16: return fir_t<_Float16>(variant, jobs, n_jobs, n_items, s);
    case LLOID_BF16: return fir_t<__bf16>(variant, jobs, n_jobs, n_items, s);
    case LLOID_F32: return fir_t<float>(variant, jobs, n_jobs, n_items, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename TS, typename TD>
static hipError_t up_t(const UpJob *jobs, int n_jobs, int64_t n_items, int r_min, hipStream_t s) {
  static_assert(4 * up_wave_lds<TS>(2) <= 64 * 1024, "within the default limit of dynamic LDS");
  k_upsample<TS, TD><<<(unsigned)n_items, 256, 4 * up_wave_lds<TS>(r_min), s>>>(jobs, n_jobs, r_min);
  return hipGetLastError();
}

hipError_t launch_up_jobs(lloid_dtype t, const UpJob *jobs, int n_jobs, int64_t n_items, int r_min, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  switch (t) {
    case LLOID_F32: return up_t<float, float>(jobs, n_jobs, n_items, r_min, s);
    case LLOID_F16: return up_t<_Float16, _Float16>(jobs, n_jobs, n_items, r_min, s);
    case LLOID_BF16: return up_t<float, __bf16>(jobs, n_jobs, n_items, r_min, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, int MT, int NT, int WM, int WN, int BK>
static hipError_t mix_v(const MixJob *jobs, int n_jobs, int64_t n_items, bool with_snr, hipStream_t s) {
  if (with_snr)
    k_mix_peak<T, MT, NT, WM, WN, BK, true><<<(unsigned)n_items, 64 * WM * WN, 0, s>>>(jobs, n_jobs);
  else
    k_mix_peak<T, MT, NT, WM, WN, BK, false><<<(unsigned)n_items, 64 * WM * WN, 0, s>>>(jobs, n_jobs);
  return hipGetLastError();
}

template <typename T>
static hipError_t mix_t(int variant, const MixJob *jobs, int n_jobs, int64_t n_items, bool with_snr, hipStream_t s) {
  switch (variant) {
    case 1: return mix_v<T, 4, 2, 2, 2, 32>(jobs, n_jobs, n_items, with_snr, s);
    case 2: return mix_v<T, 2, 2, 4, 2, 32>(jobs, n_jobs, n_items, with_snr, s);
    case 3: return mix_v<T, kMixMT, kMixNT, kMixWM, kMixWN, 32>(jobs, n_jobs, n_items, with_snr, s);
    case 4:
      // 16-bit operands: register-staged K chunks of 64 (149.5 KB of LDS, one workgroup per CU)
      if constexpr (sizeof(T) == 2) return mix_v<T, kMixMT, kMixNT, kMixWM, kMixWN, 64>(jobs, n_jobs, n_items, with_snr, s);
      else return mix_v<T, kMixMT, kMixNT, kMixWM, kMixWN, 32>(jobs, n_jobs, n_items, with_snr, s);
    default:
      // 16-bit operands: direct-to-LDS K chunks of 64, eight 64 x 128 waves.  Takes
      // the SNR series (a 48 s call of 1024 templates 485 us, 535 with the
      // register-held form) and what mix_reg_fits leaves it: a concatenated K above
      // 640, and small ones on long windows; the rest is launch_mix_reg's.
      if constexpr (sizeof(T) == 2) {
        if (with_snr) k_mix_dl<T, 4, 2, 2, 4, 64, 1, true><<<(unsigned)n_items, 512, 0, s>>>(jobs, n_jobs);
        else k_mix_dl<T, 4, 2, 2, 4, 64, 1, false><<<(unsigned)n_items, 512, 0, s>>>(jobs, n_jobs);
        return hipGetLastError();
      } else {
        return mix_v<T, kMixMT, kMixNT, kMixWM, kMixWN, 32>(jobs, n_jobs, n_items, with_snr, s);
      }
  }
}

hipError_t launch_mix_jobs(lloid_dtype t, int variant, const MixJob *jobs, int n_jobs, int64_t n_items,
                           bool with_snr, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  switch (t) {
    case LLOID_F16: return mix_t<_Float16>(variant, jobs, n_jobs, n_items, with_snr, s);
    case LLOID_BF16: return mix_t<__bf16>(variant, jobs, n_jobs, n_items, with_snr, s);
    case LLOID_F32: return mix_t<float>(variant, jobs, n_jobs, n_items, with_snr, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_peak_phase(lloid_dtype t, const MixJob *jobs, int n_jobs, int64_t n_entries, float phase_thr,
                             float trig_thr, int64_t *counts, int32_t *xi_counters, hipStream_t s) {
  if (n_entries <= 0) return hipSuccess;
  // entries per wave: 64, or so few that the 8192 waves the chip holds (256 CUs
  // x 32) get some, but a pair at least
  int per = 64;
  while (per > 2 && n_entries < (int64_t)8192 * per) per >>= 1;
  const unsigned blocks = blocks_for(n_entries, 4 * per);
  auto go = [&](auto z) {
    k_peak_phase<decltype(z)><<<blocks, 256, 0, s>>>(jobs, n_jobs, n_entries, per, phase_thr, trig_thr, counts, xi_counters);
    return hipGetLastError();
  };
  switch (t) {
    case LLOID_F16: return go(_Float16{});
    case LLOID_BF16: return go(__bf16{});
    case LLOID_F32: return go(float{});
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_trigger_jobs(const TrigJob *jobs, int n_jobs, int64_t n_elems, float thr, int64_t *counts,
                               int64_t *total, int64_t cap, lloid_trigger *out, hipStream_t s) {
  const int64_t nblk = trig_blocks(n_elems);
  if (nblk <= 0) return hipErrorInvalidValue;
  if (nblk > kTrigInline) {
    k_trigger_scan<<<1, 1024, 0, s>>>(counts, nblk, total);
    k_trigger_write<true><<<(unsigned)nblk, kTrigThreads, 0, s>>>(jobs, n_jobs, n_elems, thr, counts, cap, out, total);
  } else {
    k_trigger_write<false><<<(unsigned)nblk, kTrigThreads, 0, s>>>(jobs, n_jobs, n_elems, thr, counts, cap, out, total);
  }
  return hipGetLastError();
}

hipError_t launch_xi2(lloid_dtype t, const MixJob *jobs, int n_jobs, int64_t n_windows, int kmax, int64_t acorr_max,
                      float thr, const XiWork &xw, int n_cu, hipStream_t s) {
  if (n_windows <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)n_windows;   // one workgroup per (job, window)
  const int nks = kmax / 16;
  // the tile launch indexes the autocorrelation tables with 32-bit offsets
  if (t != LLOID_F32 && nks <= 32 && acorr_max <= INT_MAX && xw.cap > 0) {
    k_xi2_list<<<blocks, kXiThreads, 0, s>>>(jobs, n_jobs, thr, xw.units, xw.cap, xw.counters);
    // persistent: two workgroups per CU take units until the list is done
    const unsigned tb = (unsigned)std::min<int64_t>(xw.cap, 2 * (int64_t)std::max(n_cu, 1));
    const bool k16 = nks <= 16;
    if (t == LLOID_F16) {
      if (k16) k_xi2_tiles<_Float16, 16><<<tb, kXiThreads, 0, s>>>(jobs, n_jobs, xw.units, xw.cap, xw.counters);
      else k_xi2_tiles<_Float16, 32><<<tb, kXiThreads, 0, s>>>(jobs, n_jobs, xw.units, xw.cap, xw.counters);
    } else {
      if (k16) k_xi2_tiles<__bf16, 16><<<tb, kXiThreads, 0, s>>>(jobs, n_jobs, xw.units, xw.cap, xw.counters);
      else k_xi2_tiles<__bf16, 32><<<tb, kXiThreads, 0, s>>>(jobs, n_jobs, xw.units, xw.cap, xw.counters);
    }
    return hipGetLastError();
  }
  switch (t) {
    case LLOID_F16: k_xi2<_Float16><<<blocks, kXiThreads, 0, s>>>(jobs, n_jobs, thr); break;
    case LLOID_BF16: k_xi2<__bf16><<<blocks, kXiThreads, 0, s>>>(jobs, n_jobs, thr); break;
    case LLOID_F32: k_xi2<float><<<blocks, kXiThreads, 0, s>>>(jobs, n_jobs, thr); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_fft_tables(float2 *tw, float *win, hipStream_t s) {
  k_fft_tables<<<kFftMax / 256, 256, 0, s>>>(tw, win);
  return hipGetLastError();
}

template <int LG, typename TI>
static void cond_passes(const TI *x, const CondArgs &c, hipStream_t s) {
  typedef CondShape<LG> S;
  constexpr int L = S::L, nf = L / 2 + 1;
  if (c.estimate) {
    const int64_t nseg = (c.T - L) / (L / 2) + 1;
    k_cond_segment<LG, false, TI><<<blocks_for(nseg, S::SEGS), S::THREADS, 0, s>>>(x, c.T, 0, nseg, c.tw, c.win, nullptr,
                                                                                    c.parts, nullptr, nullptr, nullptr, 0);
    k_psd_mean<<<blocks_for(nf, 64), 256, 0, s>>>(c.parts, nseg, L, c.f0, c.psd, c.gain);
  } else {
    k_psd_gain<<<blocks_for(nf, 256), 256, 0, s>>>(c.psd, nf, c.f0, c.gain);
  }
  const int64_t nseg_w = (2 * (c.T - 1)) / L + 2;   // segments -1 .. floor(2 (T - 1) / L)
  const bool gating = c.gate_thr > 0.f;
  k_cond_segment<LG, true, TI><<<blocks_for(nseg_w, S::SEGS), S::THREADS, 0, s>>>(
      x, c.T, -1, nseg_w, c.tw, c.win, c.gain, nullptr, c.y, c.bad, gating ? c.loud + loud_words(c.T) : nullptr,
      gating ? loud_summary_words(c.T) : 0);
  k_overlap_add<<<blocks_for(c.T, 256 * kOverlapPer), 256, 0, s>>>(c.y, c.T, LG - 1, -1, c.gate_thr, c.out,
                                                                    gating ? c.loud : nullptr);
  if (gating) k_gate<<<blocks_for(c.T, kGateSpan), 256, 0, s>>>(c.loud, c.T, c.gate_half, c.out, c.count);
}

hipError_t launch_condition(const void *x, lloid_dtype dt, int L, const CondArgs &c, hipStream_t s) {
  auto go = [&](auto lg) {
    constexpr int LG = decltype(lg)::value;
    if (dt == LLOID_F64) cond_passes<LG>((const double *)x, c, s);
    else cond_passes<LG>((const float *)x, c, s);
  };
  switch (L) {
    case 64: go(std::integral_constant<int, 6>{}); break;
    case 128: go(std::integral_constant<int, 7>{}); break;
    case 256: go(std::integral_constant<int, 8>{}); break;
    case 512: go(std::integral_constant<int, 9>{}); break;
    case 1024: go(std::integral_constant<int, 10>{}); break;
    case 2048: go(std::integral_constant<int, 11>{}); break;
    case 4096: go(std::integral_constant<int, 12>{}); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_coincide(const lloid_trigger *a, int64_t na, const lloid_trigger *b, int64_t nb, int64_t max_dt,
                           int64_t *counts, int *bad, ResultWords *res, int64_t cap, lloid_coinc *out, uint8_t *bg_a,
                           uint8_t *bg_b, hipStream_t s) {
  const int64_t nblk = coinc_blocks(na, nb);
  k_coinc_count<<<(unsigned)nblk, kCoincThreads, 0, s>>>(a, na, b, nb, max_dt, counts, bad, bg_b);
  if (nblk > kTrigInline) {
    k_trigger_scan<<<1, 1024, 0, s>>>(counts, nblk, &res->total);
    k_coinc_write<true><<<(unsigned)nblk, kCoincThreads, 0, s>>>(a, na, b, nb, max_dt, counts, bad, res, cap, out, bg_a, bg_b);
  } else {
    k_coinc_write<false><<<(unsigned)nblk, kCoincThreads, 0, s>>>(a, na, b, nb, max_dt, counts, bad, res, cap, out, bg_a, bg_b);
  }
  return hipGetLastError();
}

hipError_t launch_sigma2(const double *mix64, int n_templates, int lsum, const double *inv_dec_per_col,
                         double *out, hipStream_t s) {
  k_sigma2<<<blocks_for(n_templates, 128), 128, 0, s>>>(mix64, n_templates, lsum, inv_dec_per_col, out);
  return hipGetLastError();
}

hipError_t launch_cast_f64(const double *src, lloid_dtype t, void *dst, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  switch (t) {
    case LLOID_F16: k_cast_f64<_Float16><<<blocks_for(n, 256), 256, 0, s>>>(src, (_Float16 *)dst, n); break;
    case LLOID_BF16: k_cast_f64<__bf16><<<blocks_for(n, 256), 256, 0, s>>>(src, (__bf16 *)dst, n); break;
    case LLOID_F32: k_cast_f64<float><<<blocks_for(n, 256), 256, 0, s>>>(src, (float *)dst, n); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_fill_u8(void *p, size_t bytes, hipStream_t s) {
  if (!bytes) return hipSuccess;
  unsigned blocks = (unsigned)std::min<size_t>((bytes + 255) / 256, 65536);
  k_fill_u8<<<blocks, 256, 0, s>>>((uint8_t *)p, bytes);
  return hipGetLastError();
}

}  // namespace lloid
