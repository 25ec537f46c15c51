// Test doubles of the HIP runtime and of the kernel launches, for CPU tests of
// the host runtime (lloid_host.cpp).  A stream is a queue of closures that runs
// when the stream is waited for, so whatever the runtime reads or writes before
// its turn, or leaves behind for work still queued, shows.  Device and pinned
// memory are heap blocks with a registry of their kinds.
#include "fake_hip.h"

#include <hip/hip_runtime.h>

#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <string>

#include "fake_state.h"
#include "lloid_internal.h"

namespace fake {

struct Block {
  size_t bytes;
  hipMemoryType type;
};
static std::map<const char *, Block> blocks;
static std::map<hipStream_t, std::deque<std::function<void()>>> queues;
State state;

static const Block *find(const void *p, size_t *left = nullptr) {
  auto it = blocks.upper_bound((const char *)p);
  if (it == blocks.begin()) return nullptr;
  --it;
  if ((const char *)p >= it->first + it->second.bytes) return nullptr;
  if (left) *left = (size_t)(it->first + it->second.bytes - (const char *)p);
  return &it->second;
}

void enqueue(hipStream_t s, std::function<void()> f) { queues[s].push_back(std::move(f)); }
size_t pending(hipStream_t s) { return queues[s].size(); }
void drain(hipStream_t s) {
  auto &q = queues[s];
  while (!q.empty()) {
    auto f = std::move(q.front());
    q.pop_front();
    f();
  }
}

// a call or launch named in state.fail_at fails, once
static bool fails(const char *name) {
  ++state.calls[name];
  if (state.fail_at != name) return false;
  if (state.fail_skip-- > 0) return false;
  state.fail_at.clear();
  return true;
}

}  // namespace fake

using fake::enqueue;
using fake::fails;

// ------------------------------------------------------------ HIP runtime

extern "C" {
hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
  *p = hipDeviceProp_t{};
  std::strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *sym) { return *p = const_cast<void *>(sym), hipSuccess; }

static hipError_t make(void **p, size_t bytes, hipMemoryType t) {
  *p = ::operator new(bytes ? bytes : 1);
  std::memset(*p, 0xa5, bytes);
  fake::blocks[(const char *)*p] = fake::Block{bytes ? bytes : 1, t};
  return hipSuccess;
}
static hipError_t drop(void *p) {
  if (!p) return hipSuccess;
  fake::blocks.erase((const char *)p);
  ::operator delete(p);
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t bytes) {
  if (fails("hipMalloc")) return hipErrorOutOfMemory;
  return make(p, bytes, hipMemoryTypeDevice);
}
hipError_t hipFree(void *p) { return drop(p); }
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned int) {
  if (fails("hipHostMalloc")) return hipErrorOutOfMemory;
  return make(p, bytes, hipMemoryTypeHost);
}
hipError_t hipHostFree(void *p) { return drop(p); }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
  const fake::Block *b = fake::find(p);
  if (!b) return hipErrorInvalidValue;
  *a = hipPointerAttribute_t{};
  a->type = b->type;
  a->devicePointer = const_cast<void *>(p);
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned int) {
  static uintptr_t next = 0x1000;
  return *s = (hipStream_t)(next += 16), hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { return fake::drain(s), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (fake::state.before_sync) {
    auto f = std::move(fake::state.before_sync);
    fake::state.before_sync = nullptr;
    f();
  }
  fake::drain(s);
  return fails("hipStreamSynchronize") ? hipErrorUnknown : hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t s) { return fake::pending(s) ? hipErrorNotReady : hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
// pageable memory: a synchronous copy in stream order; device and pinned memory: queued
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
  if (fails("hipMemcpyAsync")) return hipErrorUnknown;
  enqueue(st, [=] { std::memcpy(d, s, n); });
  if (!fake::find(d) || !fake::find(s)) fake::drain(st);
  return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, hipMemcpyKind,
                            hipStream_t st) {
  for (size_t r = 0; r < h; ++r)
    enqueue(st, [=] { std::memcpy((char *)d + r * dp, (const char *)s + r * sp, w); });
  if (!fake::find(d) || !fake::find(s)) fake::drain(st);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return *e = (hipEvent_t)1, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 0.f, hipSuccess; }
}

// ------------------------------------------------------------ kernel launches

namespace lloid {

void fir_tile_shape(lloid_dtype, int, int *bm, int *bn) { *bm = 64, *bn = 512; }
void fir_narrow_shape(int, int *bm, int *bn) { *bm = 64, *bn = 128; }
void mix_tile_shape(lloid_dtype, int, int *bm, int *bn) { *bm = *bn = 256; }

hipError_t launch_ingest(const IngestArgs &a, lloid_dtype dt, hipStream_t s) {
  if (fails("launch_ingest")) return hipErrorUnknown;
  enqueue(s, [=] {
    std::memcpy(a.tab_dst, a.tab_src, (size_t)a.tab_vecs * 16);
    for (int64_t k = 0; k < a.zero_n; ++k) a.zero[k] = 0;
    fake::state.strain.clear();
    for (int64_t k = 0; k < a.dst_len; ++k) {
      const int64_t i = a.dst_lo + k;
      double v = 0;
      if (i >= 0 && i < a.n) {
        float f;
        if (dt == LLOID_F64) std::memcpy(&v, (const char *)a.src + 8 * i, 8);
        else std::memcpy(&f, (const char *)a.src + 4 * i, 4), v = f;
      }
      a.dst[k] = (float)v * a.scale;
      if (v != v) *a.bad = 1;
      fake::state.strain.push_back(a.dst[k]);
    }
    if (fake::state.on_strain) fake::state.on_strain(fake::state.strain);
  });
  return hipSuccess;
}
hipError_t launch_trigger_jobs(const TrigJob *, int, int64_t, float, int64_t *, int64_t *total, int64_t, lloid_trigger *,
                               hipStream_t s) {
  if (fails("launch_trigger_jobs")) return hipErrorUnknown;
  const int64_t n = fake::state.triggers;
  enqueue(s, [=] { *total = n; });
  return hipSuccess;
}
hipError_t launch_fill_u8(void *p, size_t bytes, hipStream_t s) {
  enqueue(s, [=] { std::memset(p, 0, bytes); });
  return hipSuccess;
}
hipError_t launch_fft_tables(float2 *tw, float *win, hipStream_t s) {
  if (fails("launch_fft_tables")) return hipErrorUnknown;
  enqueue(s, [=] {
    std::memset((void *)tw, 0, kCondMaxLen * sizeof(float2));
    for (int i = 0; i < kCondMaxLen; ++i) win[i] = fake::kTable;
  });
  return hipSuccess;
}
hipError_t launch_condition(const void *, lloid_dtype, int, const CondArgs &c, hipStream_t s) {
  if (fails("launch_condition")) return hipErrorUnknown;
  const CondArgs a = c;
  enqueue(s, [=] {
    fake::state.table = a.win[kCondMaxLen - 1];
    for (int64_t i = 0; i < a.T; ++i) a.out[i] = 0.f;
  });
  return hipSuccess;
}
hipError_t launch_coincide(const lloid_trigger *, int64_t, const lloid_trigger *, int64_t, int64_t, int64_t *, int *,
                           ResultWords *res, int64_t, lloid_coinc *, uint8_t *, uint8_t *, hipStream_t s) {
  if (fails("launch_coincide")) return hipErrorUnknown;
  const int64_t n = fake::state.pairs;
  enqueue(s, [=] { res->total = n, res->bad = 0; });
  return hipSuccess;
}

static hipError_t plain(const char *name) { return fails(name) ? hipErrorUnknown : hipSuccess; }
hipError_t launch_decimate(DecimArgs, hipStream_t) { return plain("launch_decimate"); }
hipError_t launch_fir_jobs(lloid_dtype, int, const FirJob *, int, int64_t, hipStream_t) { return plain("launch_fir_jobs"); }
hipError_t launch_up_jobs(lloid_dtype, const UpJob *, int, int64_t, int, hipStream_t) { return plain("launch_up_jobs"); }
hipError_t launch_mix_jobs(lloid_dtype, int, const MixJob *, int, int64_t, bool, hipStream_t) {
  return plain("launch_mix_jobs");
}
hipError_t launch_mix_reg(lloid_dtype, const MixJob *, int, int64_t, hipStream_t) { return plain("launch_mix_reg"); }
hipError_t launch_peak_phase(lloid_dtype, const MixJob *, int, int64_t, float, float, int64_t *, int32_t *, hipStream_t) {
  return plain("launch_peak_phase");
}
hipError_t launch_xi2(lloid_dtype, const MixJob *, int, int64_t, int, int64_t, float, const XiWork &, int, hipStream_t) {
  return plain("launch_xi2");
}
hipError_t launch_noise(float *, int64_t, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_sigma2(const double *, int, int, const double *, double *, hipStream_t) { return hipSuccess; }
hipError_t launch_cast_f64(const double *, lloid_dtype, void *, int64_t, hipStream_t) { return hipSuccess; }

}  // namespace lloid
