// Per-process caches of what the launchers would otherwise ask the HIP runtime on every call:
// the compute-unit count of a device, and which kernels already had their dynamic-LDS limit
// raised on which device.  Both are thread-safe; after the first call on a device a launcher
// costs one hipGetDevice (a thread-local read) and a short table scan.
#include <atomic>
#include <cstdlib>
#include <mutex>
#include <utility>
#include <vector>

#include "a2d_common.hpp"

namespace a2d {
namespace {

std::atomic<int> g_cus[kMaxDevices];                       // 0 = not asked yet
std::mutex g_mu;
std::vector<std::pair<int, const void*>> g_prepared;       // (device, kernel): limit already raised
std::atomic<int> g_force_generic{-1};                      // -1 = environment not read yet

// kernel trace of the calling host thread (a2d_debug_trace)
thread_local hipEvent_t* t_trace_events = nullptr;
thread_local int t_trace_cap = 0;
thread_local int t_trace_used = 0;

thread_local const ScratchSource* t_scratch = nullptr;

}  // namespace

hipError_t device_cus(int* cus) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const bool cached = dev >= 0 && dev < kMaxDevices;
  int c = cached ? g_cus[dev].load(std::memory_order_relaxed) : 0;
  if (c <= 0) {
    e = hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    if (c <= 0) return hipErrorInvalidDevice;
    if (cached) g_cus[dev].store(c, std::memory_order_relaxed);
  }
  *cus = c;
  return hipSuccess;
}

hipError_t ensure_dynamic_lds(const void* kernel, int bytes) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const std::pair<int, const void*> key(dev, kernel);
  {
    std::lock_guard<std::mutex> lock(g_mu);
    for (const auto& p : g_prepared)
      if (p == key) return hipSuccess;
  }
  // (two threads may both get here for the same kernel: setting the attribute twice is harmless)
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(g_mu);
  g_prepared.push_back(key);
  return hipSuccess;
}

hipError_t symbol_address(const void* symbol, SymbolCache* cache, void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  void* p = cache->at[dev].load(std::memory_order_acquire);
  if (!p) {
    e = hipGetSymbolAddress(&p, symbol);
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    cache->at[dev].store(p, std::memory_order_release);   // (two first calls at once store the same address)
  }
  *out = p;
  return hipSuccess;
}

bool force_generic() {
  int v = g_force_generic.load(std::memory_order_relaxed);
  if (v < 0) {
    const char* e = getenv("A2D_FORCE_GENERIC");       // read once per process
    v = (e && e[0] == '1') ? 1 : 0;
    int expected = -1;
    if (!g_force_generic.compare_exchange_strong(expected, v)) v = expected;   // a setter came first
  }
  return v != 0;
}

void set_force_generic(bool on) { g_force_generic.store(on ? 1 : 0); }

void trace_set(hipEvent_t* events, int n) {
  t_trace_events = (events && n > 0) ? events : nullptr;
  t_trace_cap = t_trace_events ? n : 0;
  t_trace_used = 0;
}
int trace_count() { return t_trace_used; }
void trace_mark(hipStream_t s) {
  if (!t_trace_events || t_trace_used >= t_trace_cap) return;
  if (hipEventRecord(t_trace_events[t_trace_used], s) == hipSuccess) ++t_trace_used;
}

void scratch_offer(const ScratchSource* src) { t_scratch = src; }
bool scratch_offered() { return t_scratch != nullptr; }
void* scratch_get(size_t bytes) { return t_scratch ? t_scratch->get(t_scratch->ctx, bytes) : nullptr; }

int best_parts(const WalkModel& w, int cap, double merge_us, double part_us, double* time) {
  int best = 1;
  double least = walk_time(w, 1);
  for (int z = 2; z <= cap && z <= A2D_MAX_PARTS && z <= w.most; ++z) {
    const double t = walk_time(w, z) + merge_us + z * part_us;
    if (t < 0.95 * least) { best = z; least = t; }             // (a split has to be clearly better)
  }
  if (time) *time = least;
  return best;
}

double one_time(const Kind& a, const Kind& b, int slots, bool uneven, double tail) {
  if (a.n + b.n <= slots) return a.most;
  if (uneven) {                                            // longest first
    const double even = (a.n * a.mean + b.n * b.mean) / slots + tail * b.mean;
    const double late = b.most > a.most ? a.n / slots * a.mean + b.most : a.most;   // (or the longest of the second kind)
    return even > late ? even : late;
  }
  // whole turns of the first kind; then the slots it leaves free in its last turn, and the others, take the second
  const int64_t rest = a.n % slots, free = slots - rest;
  double u = (double)(a.n / slots) * a.most, v = rest ? u + a.most : u, end = v;
  for (int64_t left = b.n; left > 0;) {
    double& t = u <= v || !rest ? u : v;
    left -= &t == &u ? free : rest;
    t += b.most;
    if (t > end) end = t;
  }
  return end;
}

double dealt_time(const Kind& a, const Kind& b, int slots, bool uneven, double tail) {
  if (a.n + b.n <= slots) return a.most;
  const int engines = slots < kEngineSlots ? 1 : slots / kEngineSlots, each = slots / engines;
  double worst = 0;
  for (int i = 0; i < engines; ++i) {                      // workgroups i, i + engines, ..
    const int64_t na = (a.n - i + engines - 1) / engines, nb = (a.n + b.n - i + engines - 1) / engines - na;
    const double t = one_time(Kind{na, a.mean, a.most}, Kind{nb, b.mean, b.most}, each, uneven, tail);
    if (t > worst) worst = t;
  }
  return worst;
}

double mean_visible_keys(const a2d_tile_desc& d, const SegList& g, double seen[8]) {
  double mean = 0;
  for (int i = 0; i < 8; ++i) {
    seen[i] = (double)visible_keys(d, g, (15 - 2 * i) * (int64_t)d.nq / 16);
    mean += seen[i] / 8;
  }
  return mean;
}

void plan_fwd(const a2d_tile_desc& d, SegList* g, bool may_split, int cus) {
  const int64_t part = (int64_t)d.heads * d.nq * (d.hdim + 2) * sizeof(float);
  const int64_t cap = may_split ? (int64_t)kSplitBytes / part : 1;
  if (d.dtype == A2D_F32) plan_fwd_f32(d, g, cus, cap < 1 ? 1 : (int)cap);
  else plan_fwd_mfma(d, g, cus, cap < 1 ? 1 : (int)cap);
}

namespace {
void add(Route* r, const char* kernel) { r->kernel[r->kernels++] = kernel; }
}  // namespace

void route_fwd(const a2d_tile_desc& d, const SegList& g, Route* r) {
  *r = Route{};
  const bool f32 = d.dtype == A2D_F32, small = !f32 && g.form >= 3;
  static const int kRows[2][5] = {{256, 128, 128, 32, 64}, {16, 32, 0, 0, 0}};     // of the forms
  static const int kLanes[2][5] = {{1, 2, 1, 8, 4}, {4, 4, 0, 0, 0}};
  add(r, f32 ? "fwd_f32_kernel" : small ? "fwd_small_kernel" : "fwd_mfma_kernel");
  r->rows = kRows[f32][g.form];
  r->lanes = kLanes[f32][g.form];
  r->parts_q = g.parts;
  r->parts_kv = 1;
  r->phased = !f32 && g.phased;
}

void route_bwd(const a2d_tile_desc& d, const BwdParts& p, Route* r) {
  *r = Route{};
  r->parts_q = p.q;
  r->parts_kv = p.kv;
  if (d.dtype == A2D_F32) {
    if (p.delta) add(r, "delta_kernel");
    add(r, "bwd_f32_kernel");
    r->rows = r->keys = 16;
    r->lanes = 4;
    return;
  }
  if (p.small) {
    add(r, "bwd_small_kernel");
    r->apart = p.small > 1;
    r->rows = r->keys = 32;
    r->lanes = 8;
    return;
  }
  const char* const kv = p.wide ? "bwd_dkdv_wide_kernel" : "bwd_dkdv_kernel";
  if (p.one || p.keep_ds) {
    if (p.wide || p.keep_ds) add(r, "delta_kernel");
    add(r, p.one ? "bwd_one_kernel" : kv);
    if (!p.one) add(r, "bwd_dq_ds_kernel");
  } else {
    add(r, "bwd_dq_kernel");
    add(r, kv);
  }
  r->rows = p.form == 0 ? 256 : 128;
  r->lanes = p.form == 1 ? 2 : 1;
  r->keys = p.wide ? 256 : 128;
}

int64_t visible_keys(const a2d_tile_desc& d, const SegList& g, int64_t i) {
  if (!d.causal) return d.nkv;
  int64_t n = 0;
  for (int s = 0; s < g.n; ++s) {
    const int64_t v = i + g.seg[s].rel + 1;
    n += v <= 0 ? 0 : (v < g.seg[s].rows ? v : g.seg[s].rows);
  }
  return n;
}

}  // namespace a2d
