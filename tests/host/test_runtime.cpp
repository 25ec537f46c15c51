// CPU tests of the host runtime (lloid_host.cpp) over the test doubles of
// fake_hip.cpp; built and run by tests/test_host_runtime.py.
#include <cmath>
#include <cstdio>
#include <cstring>

#include "fake_state.h"
#include "lloid_internal.h"

using namespace lloid;

static int g_fail = 0;
#define CHECK(cond)                                              \
  do {                                                           \
    if (!(cond)) {                                               \
      std::printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #cond); \
      ++g_fail;                                                  \
    }                                                            \
  } while (0)

namespace {

hipStream_t caller_stream() {
  hipStream_t s;
  (void)hipStreamCreateWithFlags(&s, 0);
  return s;
}

lloid_ctx *make_ctx(hipStream_t s) {
  lloid_ctx *c = nullptr;
  CHECK(lloid_ctx_create(0, s, &c) == LLOID_OK);
  return c;
}

lloid_bank *make_bank(lloid_ctx *c, int templates, int basis, int levels, int f0 = 1024,
                      lloid_dtype ct = LLOID_F16) {
  std::vector<double> u((size_t)basis * 64, 0.1), m((size_t)2 * templates * basis, 0.1);
  std::vector<lloid_slice> sl;
  for (int k = 0; k < levels; ++k) {
    lloid_slice s{};
    s.rate_hz = f0 >> k;
    s.start_tap = 128 * k;
    s.n_taps = 64;
    s.n_basis = basis;
    s.basis = u.data();
    s.mixing = m.data();
    sl.push_back(s);
  }
  lloid_bank_desc d{};
  d.full_rate_hz = f0;
  d.n_templates = templates;
  d.n_slices = levels;
  d.slices = sl.data();
  d.compute = ct;
  lloid_bank *b = nullptr;
  CHECK(lloid_bank_create(c, &d, &b) == LLOID_OK);
  return b;
}

bool holds(const std::vector<float> &got, int64_t n, float v) {
  if ((int64_t)got.size() != n) return false;
  for (float x : got)
    if (x != v) return false;
  return true;
}

// The strain is read when the context's stream comes to the call, whatever the
// kind of memory, the block's length and the entry point: work queued there
// before may still be filling the buffer.
void strain_in_stream_order() {
  hipStream_t s = caller_stream();
  lloid_ctx *c = make_ctx(s);
  lloid_bank *b = make_bank(c, 4, 16, 1);
  for (int64_t n : {100, 8192, 100000})
    for (int kind = 0; kind < 3; ++kind)
      for (int noalloc = 0; noalloc < 2; ++noalloc)
        for (int off = 0; off < 2; ++off) {     // a buffer that is not aligned to its samples
          const size_t bytes = (size_t)n * 4 + 8;
          void *p = nullptr;
          if (kind == 0) p = std::malloc(bytes);
          else CHECK((kind == 1 ? hipHostMalloc(&p, bytes, 0) : hipMalloc(&p, bytes)) == hipSuccess);
          char *x = (char *)p + 2 * off;
          for (int64_t i = 0; i < n; ++i) std::memset(x + 4 * i, 0, 4);
          fake::enqueue(s, [=] {
            const float v = 3.f;
            for (int64_t i = 0; i < n; ++i) std::memcpy(x + 4 * i, &v, 4);
          });
          lloid_trigger t[4];
          int64_t nt = 0;
          const lloid_status r =
              noalloc ? lloid_filter_noalloc(b, 0, x, LLOID_F32, n, nullptr, t, 4, &nt, nullptr)
                      : lloid_filter(b, 0, x, LLOID_F32, n, nullptr, t, 4, &nt, nullptr, nullptr);
          CHECK(r == LLOID_OK);
          CHECK(holds(fake::state.strain, n, 3.f));
          if (kind == 0) std::free(p);
          else (void)(kind == 1 ? hipHostFree(p) : hipFree(p));
        }
  lloid_bank_destroy(b);
  lloid_ctx_destroy(c);
}

// A call of the allocation-free form shares nothing with the other calls of the
// context: one that comes between another's launches and its wait leaves that
// one's strain, tables and result words alone, and the other way round.
void noalloc_calls_overlap_others() {
  lloid_ctx *c = make_ctx(nullptr);
  lloid_bank *b = make_bank(c, 4, 16, 1);
  const int64_t n = 3000;
  const std::vector<float> one((size_t)n, 1.f), two((size_t)n, 2.f);
  lloid_trigger t[8], t2[8];
  int64_t nt = 0, nt2 = 0;
  lloid_coinc pairs[8];
  auto filter = [&](const std::vector<float> &x, lloid_trigger *t, int64_t *nt, int triggers, bool noalloc) {
    fake::state.triggers = triggers;
    CHECK((noalloc ? lloid_filter_noalloc(b, 0, x.data(), LLOID_F32, n, nullptr, t, 8, nt, nullptr)
                   : lloid_filter(b, 0, x.data(), LLOID_F32, n, nullptr, t, 8, nt, nullptr, nullptr)) == LLOID_OK);
  };
  filter(one, t, &nt, 0, false);   // the context's workspace has its size
  for (int inner = 0; inner < 2; ++inner) {
    std::vector<std::vector<float>> seen;
    fake::state.on_strain = [&](const std::vector<float> &x) { seen.push_back(x); };
    fake::state.before_sync = [&] { filter(two, t2, &nt2, 5, inner == 1); };
    filter(one, t, &nt, 3, inner == 0);
    CHECK(nt == 3 && nt2 == 5);
    CHECK(seen.size() == 2 && holds(seen[0], n, 1.f) && holds(seen[1], n, 2.f));
    fake::state.on_strain = nullptr;
  }
  int64_t np = 0;
  fake::state.pairs = 7;
  fake::state.before_sync = [&] { filter(two, t2, &nt2, 5, true); };
  std::memset(t, 0, sizeof t);
  CHECK(lloid_coincide(c, t, 8, t, 8, 3, pairs, 8, &np, nullptr) == LLOID_OK);
  CHECK(np == 7 && nt2 == 5);
  lloid_bank_destroy(b);
  lloid_ctx_destroy(c);
}

// A call that fails between its first launch and its wait leaves nothing queued.
void failed_calls_leave_nothing_queued() {
  hipStream_t s = caller_stream();
  lloid_ctx *c = make_ctx(s);
  lloid_bank *b = make_bank(c, 4, 16, 3);
  const int64_t n = 60000;   // an upload of its own
  std::vector<float> x((size_t)n, 1.f), out((size_t)n);
  std::vector<double> psd(129, 1.0);
  lloid_trigger t[8] = {};
  lloid_coinc pairs[8];
  uint8_t bg[16];
  lloid_condition_opts co{};
  co.seg_len = 256;
  auto call = [&](int which) -> lloid_status {
    int64_t k = 0;
    switch (which) {
      case 0: return lloid_filter(b, 0, x.data(), LLOID_F32, n, nullptr, t, 8, &k, nullptr, nullptr);
      case 1: return lloid_filter_noalloc(b, 0, x.data(), LLOID_F32, 900, nullptr, t, 8, &k, nullptr);
      case 2: co.psd = nullptr; return lloid_condition(c, 1024, x.data(), LLOID_F32, n, &co, out.data(), psd.data(), &k);
      case 3: co.psd = psd.data(); return lloid_condition(c, 1024, x.data(), LLOID_F32, n, &co, out.data(), nullptr, &k);
      default: return lloid_coincide(c, t, 8, t, 8, 3, pairs, 8, &k, bg);
    }
  };
  fake::state.triggers = 3;
  fake::state.pairs = 3;
  for (int which = 0; which < 5; ++which) CHECK(call(which) == LLOID_OK);   // workspaces have their sizes
  int failed = 0;
  for (const char *name : {"launch_ingest", "launch_decimate", "launch_fir_jobs", "launch_up_jobs", "launch_mix_jobs",
                           "launch_mix_reg", "launch_peak_phase", "launch_trigger_jobs", "launch_condition",
                           "launch_coincide", "hipMemcpyAsync"})
    for (int which = 0; which < 5; ++which)
      for (int skip = 0; skip < 6; ++skip) {
        fake::state.fail_at = name;
        fake::state.fail_skip = skip;
        const lloid_status r = call(which);
        const bool hit = fake::state.fail_at.empty();
        fake::state.fail_at.clear();
        CHECK(hit ? r != LLOID_OK : r == LLOID_OK);
        CHECK(fake::pending(s) == 0);
        failed += hit;
        CHECK(call(which) == LLOID_OK);
      }
  CHECK(failed >= 30);
  lloid_bank_destroy(b);
  lloid_ctx_destroy(c);
}

// A conditioning call whose transform tables could not be made leaves none
// behind: the next one makes them.
void transform_tables_are_whole() {
  lloid_ctx *c = make_ctx(nullptr);
  const int64_t n = 600;
  std::vector<float> x((size_t)n, 1.f), out((size_t)n);
  lloid_condition_opts co{};
  co.seg_len = 256;
  for (const char *name : {"launch_fft_tables", "hipMalloc"}) {
    const bool alloc = std::strcmp(name, "hipMalloc") == 0;
    if (alloc) lloid_ctx_destroy(c), c = make_ctx(nullptr);
    fake::state.table = 0.f;
    fake::state.fail_skip = alloc ? 1 : 0;   // the workspace, then the tables
    fake::state.fail_at = name;
    CHECK(lloid_condition(c, 1024, x.data(), LLOID_F32, n, &co, out.data(), nullptr, nullptr) != LLOID_OK);
    CHECK(fake::state.fail_at.empty());
    CHECK(lloid_condition(c, 1024, x.data(), LLOID_F32, n, &co, out.data(), nullptr, nullptr) == LLOID_OK);
    CHECK(fake::state.table == fake::kTable);
  }
  lloid_ctx_destroy(c);
}

// What the allocation-free call takes of its scratch with one window per chunk
// has not grown past what callers have sized their blocks for: the longest block
// whose strain levels, peak tables, operands, low-rate buffers and tables (of
// 120, 112, 240 and 88 bytes an entry) come to the scratch's size is accepted.
void noalloc_accepts_what_fits() {
  lloid_ctx *c = make_ctx(nullptr);
  const int f0 = 1024, win_len = 4, F = 600;
  for (int levels : {1, 3, 8}) {
    lloid_bank *b = make_bank(c, F, 16, levels, f0);
    auto need = [&](int64_t W) {
      const int64_t n = W * win_len;
      size_t bytes = 0, n_fir = 0, n_up = 0;
      auto add = [&](size_t cnt, size_t sz) { bytes = (size_t)round_up((int64_t)bytes, 256) + cnt * sz; };
      Range sup{0, n};
      for (int k = 0; k < levels; ++k, sup = halo_up(sup)) add((size_t)sup.size(), 4);
      const size_t tab = (size_t)F * W;
      for (size_t sz : {4, 8, 4, 4, 4, 4, 8}) add(tab, sz);
      const int64_t ops = std::min<int64_t>(n, win_len + 1) + 2;
      add((size_t)ops * b->kld, 2);
      for (const auto &sl : b->slices) {
        ++n_fir;
        if (sl.level > 0)
          for (int64_t ld : low_ld(ops, sl.level)) add((size_t)sl.lp * ld, 2), ++n_up;
      }
      add((size_t)trig_blocks((int64_t)tab) + 2, 8);
      add(1, 4);
      add(0, sizeof(XiUnit));
      add(2, 4);
      add(8, sizeof(lloid_trigger));
      add((size_t)W * (n_fir * 120 + n_up * 112 + 240 + 64 * (3 + kMaxHops)) + 88 + 256, 1);
      return bytes;
    };
    int64_t lo = 1, hi = int64_t(1) << 24;
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) / 2;
      (need(mid) <= (size_t)LLOID_NOALLOC_SCRATCH_BYTES ? lo : hi) = mid;
    }
    void *x = nullptr;
    CHECK(hipMalloc(&x, (size_t)lo * win_len * 4) == hipSuccess);
    std::memset(x, 0, (size_t)lo * win_len * 4);
    lloid_trigger_opts o{};
    o.window_num = win_len;
    o.window_den = f0;
    o.threshold = 4.f;
    lloid_trigger t[8];
    int64_t nt = 0;
    const lloid_status r = lloid_filter_noalloc(b, 0, x, LLOID_F32, lo * win_len, &o, t, 8, &nt, nullptr);
    CHECK(r == LLOID_OK);
    if (r != LLOID_OK) std::printf("%lld windows: %s\n", (long long)lo, lloid_last_error());
    (void)hipFree(x);
    lloid_bank_destroy(b);
  }
  lloid_ctx_destroy(c);
}

// The two mixing launches split one table: the register-held form's jobs come
// last, each part longest K first, and the items of each launch are numbered
// from 0 in the order of its jobs.
void mixing_forms_split_the_table() {
  // beyond K = 640 and, on long windows, below K = 128 the direct-to-LDS form is used
  CHECK(mix_reg_fits(640, 1 << 20) && !mix_reg_fits(672, 1));
  CHECK(mix_reg_fits(32, 512) && !mix_reg_fits(32, 1024) && mix_reg_fits(64, 1024) && !mix_reg_fits(64, 2048));
  CHECK(mix_reg_fits(96, 4096) && !mix_reg_fits(96, 16384) && mix_reg_fits(128, 1 << 20));
  const int ks[] = {96, 672, 32, 640, 64, 128, 1024, 160};
  for (int64_t win_len : {33, 1024, 2048, 100000})
    for (lloid_dtype ct : {LLOID_F16, LLOID_F32})
      for (int variant : {0, 3}) {
        const TileShapes ts(ct, 0, variant);
        std::vector<FirJob> fj;
        std::vector<UpJob> uj[kMaxHops];
        std::vector<MixJob> mj;
        for (int k : ks) {
          MixJob m{};
          m.kcat = k;
          m.kld = (int)round_up(k, 64);
          m.rows = 512;
          m.n_templates = 200;
          m.nw = 11;
          m.win_p = win_len;
          m.win_q = 1;
          m.n_rtiles = (int)ceil_div(m.rows, ts.mbm);
          mj.push_back(m);
        }
        StageItems n;
        number_jobs(ct, fj, uj, mj, win_len, ts, 256, n);
        const int dl = (int)mj.size() - n.n_mix_reg;
        int64_t next[2] = {0, 0}, e = 0;
        for (int i = 0; i < (int)mj.size(); ++i) {
          const bool r = mix_reg_job(ct, variant, mj[i]);
          CHECK(r == (i >= dl));
          CHECK(i == 0 || i == dl || mj[i - 1].kcat >= mj[i].kcat);
          CHECK(mj[i].item0 == next[r]);
          const int64_t units = r ? ceil_div(mj[i].nw * mj[i].tpw, mj[i].run) : mj[i].nw * mj[i].parts;
          next[r] += units >= 8 ? ceil_div(units, 8) * 8 * mj[i].n_rtiles : round_up(units * mj[i].n_rtiles, 8);
          CHECK(mj[i].e0 == e);
          e += mj[i].nw * mj[i].n_templates;
        }
        CHECK(n.mix == next[0] && n.mix_reg == next[1] && n.entries == e);
      }
}

}  // namespace

int main() {
  mixing_forms_split_the_table();
  noalloc_accepts_what_fits();
  strain_in_stream_order();
  noalloc_calls_overlap_others();
  failed_calls_leave_nothing_queued();
  transform_tables_are_whole();
  std::printf(g_fail ? "%d checks failed\n" : "ok\n", g_fail);
  return g_fail != 0;
}
