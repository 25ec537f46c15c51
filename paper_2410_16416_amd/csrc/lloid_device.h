// Device code shared by the kernel files: MFMA operand types, buffer
// resources, work-item lookup and the window-peak keys.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lloid_internal.h"

namespace lloid {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------- MFMA ops
// Operand type T: K per instruction (KS), elements per lane per operand (VEC).
// Lane l of a 32x32xKS instruction supplies row/column l % 32 and the VEC
// consecutive k values starting at (l / 32) * VEC; the 32x32 FP32 result puts
// rows 8 (r/4) + 4 (l/32) + r%4, r = 0..15, of column l % 32 in lane l.
template <typename T> struct Op;

template <> struct Op<_Float16> {
  static constexpr int KS = 16, VEC = 8;
  typedef half8 vec;
  static __device__ __forceinline__ f32x16 mfma(vec a, vec b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ _Float16 cvt(float v) { return (_Float16)v; }
  static __device__ __forceinline__ float tof(_Float16 v) { return (float)v; }
};

template <> struct Op<__bf16> {
  static constexpr int KS = 16, VEC = 8;
  typedef bf16x8 vec;
  static __device__ __forceinline__ f32x16 mfma(vec a, vec b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ __bf16 cvt(float v) { return (__bf16)v; }
  static __device__ __forceinline__ float tof(__bf16 v) { return (float)v; }
};

template <> struct Op<float> {
  static constexpr int KS = 2, VEC = 1;
  typedef float vec;
  static __device__ __forceinline__ f32x16 mfma(vec a, vec b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ float cvt(float v) { return v; }
  static __device__ __forceinline__ float tof(float v) { return v; }
};

// Job owning flat work item `item`: the last job with item0 <= item.
template <typename J>
__device__ __forceinline__ int find_job(const J *__restrict__ jobs, int n_jobs, int64_t item) {
  int lo = 0, hi = n_jobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].item0 <= item) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Buffer resource over `bytes` bytes from `base`: loads past the end (or at
// negative offsets, which wrap to huge unsigned ones) return zero in hardware.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, int64_t bytes) {
  const int nb = bytes <= 0 ? 0 : (bytes > 0x7ffffff0 ? 0x7ffffff0 : (int)bytes);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, nb, 0x00020000);
}

struct VN {
  float v;
  int n;
};

// A window peak as one ordered word: |z|^2 (its bits order as integers, it is
// not negative), then the complement of the sample (relative to the window's
// start), so that the largest word is the largest |z|^2 at its lowest
// sample.  0: no sample compared greater than the initial -1.
__device__ __forceinline__ uint64_t peak_key(VN p) {
  return p.v < 0.f ? 0 : ((uint64_t)__float_as_uint(p.v) << 32) | (uint32_t)~p.n;
}

__device__ __forceinline__ VN peak_of_key(uint64_t k) {
  return k ? VN{__uint_as_float((uint32_t)(k >> 32)), (int)~(uint32_t)k} : VN{-1.f, 0x7fffffff};
}

// A workgroup's peak of template i in window w: stored, or combined with the
// other parts' (an integer maximum, so the order does not matter).
__device__ __forceinline__ void put_peak(const MixJob &jb, int64_t i, int64_t w, VN p) {
  uint64_t *k = (uint64_t *)jb.peak_n + (i * jb.ld_peak + (w - jb.w_base));
  if (jb.parts == 1) *k = peak_key(p);
  else if (p.v >= 0.f) atomicMax((unsigned long long *)k, (unsigned long long)peak_key(p));
}

}  // namespace lloid
