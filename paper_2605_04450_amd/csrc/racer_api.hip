// C-ABI layer: argument checks, host bookkeeping, workspaces, kernel launches.
// Declarations and their semantics are in include/racer_pool.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <new>
#include <string>
#include <vector>

#include "../../include/racer_pool.h"  // also fixes RACER_NOALLOC_MAX_*
#include "kernels.h"
#include "pool_host.h"
#include "alpha_ctl.h"

namespace {

thread_local std::string g_last_error;

int32_t hip_fail(hipError_t e, const char* what) {
  g_last_error = std::string(what) + ": " + hipGetErrorString(e);
  return RACER_EHIP;
}

#define HIP_TRY(expr)                                   \
  do {                                                  \
    hipError_t _e = (expr);                             \
    if (_e != hipSuccess) return hip_fail(_e, #expr);   \
  } while (0)

bool is_pow2(uint64_t x) { return x && !(x & (x - 1)); }

// Tests of the error paths name the call that is to fail once in the environment (RACER_FAULT_INJECT=split); the
// variable is cleared by the call that honours it.  Nothing on the GPU is made to fail: the call returns before it
// queues its device work.
bool fault_injected(const char* what) {
  const char* v = std::getenv("RACER_FAULT_INJECT");
  if (!v || std::strcmp(v, what) != 0) return false;
  unsetenv("RACER_FAULT_INJECT");
  return true;
}

// Device memory for metadata and workspaces.  With `zero` the memory is cleared by a fill kernel on `stream`,
// the stream whose later kernels use it (a clear on the null stream is not ordered with a non-blocking stream).
template <typename T>
int32_t dev_alloc(T** p, uint64_t count, bool zero, hipStream_t stream) {
  *p = nullptr;
  if (count == 0) count = 1;
  const uint64_t bytes = (count * sizeof(T) + 3) & ~3ull;  // cleared in 32-bit words
  HIP_TRY(hipMalloc(reinterpret_cast<void**>(p), bytes));
  if (zero) HIP_TRY(racer::launch_fill_u32(reinterpret_cast<uint32_t*>(*p), bytes / 4, 0u, stream));
  return RACER_OK;
}

// Pinned staging that is written by the host and copied to the device (or read by a kernel) asynchronously;
// two buffers alternate so a call only ever waits for the copy issued two calls earlier.
struct Staging {
  uint8_t* buf[2] = {nullptr, nullptr};
  hipEvent_t done[2] = {nullptr, nullptr};
  uint64_t cap[2] = {0, 0};
  bool pending[2] = {false, false};
  int next = 0;
  uint64_t allocs = 0;  // pinned (re)allocations so far

  // both buffers at least `bytes` large, so that no later acquire of up to that size allocates
  int32_t reserve(uint64_t bytes) {
    for (int k = 0; k < 2; ++k) {
      if (!done[k]) HIP_TRY(hipEventCreateWithFlags(&done[k], hipEventDisableTiming));
      if (cap[k] >= bytes) continue;
      if (pending[k]) {
        HIP_TRY(hipEventSynchronize(done[k]));
        pending[k] = false;
      }
      if (buf[k]) HIP_TRY(hipHostFree(buf[k]));
      buf[k] = nullptr;
      cap[k] = 0;
      HIP_TRY(hipHostMalloc(reinterpret_cast<void**>(&buf[k]), bytes, hipHostMallocCoherent));
      cap[k] = bytes;
      ++allocs;
    }
    return RACER_OK;
  }

  int32_t acquire(uint64_t bytes, uint8_t** out, int* which) {
    const int k = next;
    next ^= 1;
    if (pending[k]) {
      HIP_TRY(hipEventSynchronize(done[k]));
      pending[k] = false;
    }
    if (cap[k] < bytes) {
      if (buf[k]) HIP_TRY(hipHostFree(buf[k]));
      buf[k] = nullptr;
      cap[k] = 0;
      const uint64_t want = std::max<uint64_t>(bytes * 2, 1 << 16);
      HIP_TRY(hipHostMalloc(reinterpret_cast<void**>(&buf[k]), want, hipHostMallocCoherent));
      cap[k] = want;
      ++allocs;
    }
    if (!done[k]) HIP_TRY(hipEventCreateWithFlags(&done[k], hipEventDisableTiming));
    *out = buf[k];
    *which = k;
    return RACER_OK;
  }
  int32_t mark(int which, hipStream_t s) {
    HIP_TRY(hipEventRecord(done[which], s));
    pending[which] = true;
    return RACER_OK;
  }
  void release() {
    for (int k = 0; k < 2; ++k) {
      if (pending[k]) (void)hipEventSynchronize(done[k]);
      if (buf[k]) (void)hipHostFree(buf[k]);
      if (done[k]) (void)hipEventDestroy(done[k]);
      buf[k] = nullptr;
      done[k] = nullptr;
      pending[k] = false;
      cap[k] = 0;
    }
  }
};

// ---- work space of emb_lookup_noalloc -----------------------------------------------------------------------
// One array per GPU, part of the library's code object, alive until the process ends.  It holds the miss path's
// lists for up to kNoallocMaxLookups lookups whose rows add up to at most kNoallocStagingBytes.  In host code the
// array's name is only a handle for hipGetSymbolAddress: the address that kernels and fills take is the one
// that call returns for the current device, kept in g_scratch_ptr.
constexpr uint64_t kNoallocMaxLookups = RACER_NOALLOC_MAX_LOOKUPS;
constexpr uint64_t kNoallocStagingBytes = RACER_NOALLOC_MAX_ROW_BYTES_TOTAL;
constexpr uint64_t kNoallocHash = 2 * kNoallocMaxLookups;  // slots of the dedupe table and of the set-chain heads
constexpr uint64_t align256(uint64_t x) { return (x + 255) & ~255ull; }
// control words, dedupe table and chain heads come first, one after the other for the table size of the call, so that
// one fill clears them
constexpr uint64_t kOffHents = 256;
constexpr uint64_t kClearBytes = sizeof(racer::HashEnt) + sizeof(unsigned long long);  // per table slot
constexpr uint64_t kOffSegCnt = kOffHents + align256(kClearBytes * kNoallocHash);   // u32 [lookups / kMinStretch + 2]
constexpr uint64_t kOffDefList = kOffSegCnt + align256(4 * (kNoallocMaxLookups / racer::kMinStretch + 2));  // u32 [lookups]
constexpr uint64_t kOffLoc = kOffDefList + align256(4 * kNoallocMaxLookups);        // i64 [lookups]
constexpr uint64_t kOffHslot = kOffLoc + align256(8 * kNoallocMaxLookups);          // u32 [hash]
constexpr uint64_t kOffRec = kOffHslot + align256(4 * kNoallocHash);                // uint4 [lookups]
constexpr uint64_t kOffWay = kOffRec + align256(16 * kNoallocMaxLookups);           // i32 [lookups]
constexpr uint64_t kOffStaging = kOffWay + align256(4 * kNoallocMaxLookups);
constexpr uint64_t kScratchBytes = kOffStaging + kNoallocStagingBytes;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
uint8_t* g_scratch_ptr[kMaxDevices] = {};

// address of the current device's copy of `scratch` (looked up once per device)
int32_t scratch_address(uint8_t** out) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return RACER_EINVAL;
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return RACER_EHIP;
    g_scratch_ptr[dev] = static_cast<uint8_t*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return RACER_OK;
}

}  // namespace

// Host-side arrays of prepare_step, kept from call to call for their memory.
struct StepScratch {
  racer::AttnSchedule attn;
  std::vector<racer::ReqDev> reqs;
  std::vector<racer::RowTile> row_tiles;
  std::vector<racer::F32Tile> f32_tiles;
};

struct racer_pool {
  racer::HostPool host;
  racer_pool_cfg cfg;
  uint8_t* base = nullptr;
  uint64_t bytes = 0, page_size = 0;
  bool device = false;
  uint32_t* d_tags = nullptr;
  uint32_t* d_stamps = nullptr;
  int32_t* d_emb_pages = nullptr;
  unsigned long long* d_counters = nullptr;
  const uint8_t* d_table = nullptr;
  // every table behind the pool (the first is pool_create's); the device copy exists once a second one was added
  std::vector<racer::TableDesc> tables;
  racer::TableDesc* d_tables = nullptr;
  Staging stage;
  uint32_t batch = 0;
  uint64_t ws_allocs = 0;  // device work-space (re)allocations so far (pool_reserve keeps later calls from adding any)
  hipStream_t last_stream = nullptr;
  // miss-path workspace, grown on demand
  uint64_t ws_cap = 0;
  racer::MissWs ws{};
  // hstu workspace
  uint64_t hw_slot = 0;  // bytes of each of the six activation matrices of a step
  uint8_t* hw_buf = nullptr;
  uint64_t hl_cap = 0;
  uint8_t* hl_dev = nullptr;
  uint64_t hp_cap = 0;  // fp32 partial outputs of split attention items
  uint8_t* hp_dev = nullptr;
  Staging hstage;
  StepScratch step;
  uint32_t step_epoch = 0;  // number of the step: a request with unordered timestamps is marked with it
  uint32_t* ts_marks = nullptr;
  uint64_t ts_marks_cap = 0;
  // optional per-kernel-class timing with events on the caller's stream
  struct ProfMark { hipEvent_t a, b; int kind; };
  bool prof_on = false;
  std::vector<ProfMark> prof;
  std::vector<hipEvent_t> prof_spare;

  racer_pool(uint64_t n_pages, const racer_pool_cfg& c, uint32_t spp) : host(n_pages, c.page_tokens, spp, c.w_max), cfg(c) {}

  racer::EmbView view() const {
    racer::EmbView v{};
    v.base = base;
    v.page_size = page_size;
    v.row_bytes = cfg.row_bytes;
    v.spp = host.spp();
    v.w_max = cfg.w_max;
    v.elem = cfg.elem;
    v.sets = static_cast<uint32_t>(host.sets());
    v.layer_pages = static_cast<uint32_t>(host.layer_pages());
    v.full_ways = static_cast<uint32_t>(host.n_emb() / host.layer_pages());
    v.part_sets = static_cast<uint32_t>((host.n_emb() % host.layer_pages()) * host.spp());
    v.tags = d_tags;
    v.stamps = d_stamps;
    v.emb_pages = d_emb_pages;
    v.table = d_table;
    v.rows = tables.empty() ? cfg.rows : tables.back().base + tables.back().rows;
    v.tables = tables.size() > 1 ? d_tables : nullptr;
    v.n_tables = static_cast<uint32_t>(tables.size());
    v.counters = d_counters;
    return v;
  }
};

struct racer_hstu {
  racer_hstu_cfg cfg;
  racer_hstu_weights w;
  // bf16 models: half-precision copies of W1 and W2, as operand fragments for the fused layer halves, else output-major
  void* w1t = nullptr;
  void* w2t = nullptr;
  float* pos_s = nullptr;   // bf16 models: pos and time tables times log2(e), as the attention kernel wants them
  float* time_s = nullptr;
};

namespace {

// Bracket one launch (or a fixed group of launches) with events when timing is enabled.
struct ProfScope {
  racer_pool* p;
  hipStream_t s;
  bool live = false;
  ProfScope(racer_pool* pool, int kind, hipStream_t stream) : p(pool), s(stream) {
    if (!p->prof_on) return;
    hipEvent_t ev[2] = {nullptr, nullptr};
    for (hipEvent_t& e : ev) {
      if (!p->prof_spare.empty()) {
        e = p->prof_spare.back();
        p->prof_spare.pop_back();
      } else if (hipEventCreate(&e) != hipSuccess) {
        return;
      }
    }
    if (hipEventRecord(ev[0], s) != hipSuccess) return;
    p->prof.push_back({ev[0], ev[1], kind});
    live = true;
  }
  ~ProfScope() {
    if (live) (void)hipEventRecord(p->prof.back().b, s);
  }
};

void free_miss_ws(racer_pool* p) {
  racer::MissWs& w = p->ws;
  (void)hipFree(w.any); (void)hipFree(w.seg_cnt); (void)hipFree(w.def_list); (void)hipFree(w.loc); (void)hipFree(w.hents);
  (void)hipFree(w.hslot_u); (void)hipFree(w.heads); (void)hipFree(w.rec); (void)hipFree(w.u_way); (void)hipFree(w.staging);
  p->ws = racer::MissWs{};
  p->ws_cap = 0;
}

int32_t ensure_miss_ws(racer_pool* p, uint64_t n, hipStream_t stream) {
  if (n <= p->ws_cap) return RACER_OK;
  if (p->ws_cap) {
    HIP_TRY(hipStreamSynchronize(p->last_stream));
    free_miss_ws(p);
  }
  const uint64_t cap = std::max<uint64_t>(n, 1024);
  uint64_t hsize = 2048;
  while (hsize < 2 * cap) hsize <<= 1;
  p->ws_allocs += 1;
  racer::MissWs& w = p->ws;
  int32_t rc;
  if ((rc = dev_alloc(&w.any, 64, true, stream))) return rc;
  if ((rc = dev_alloc(&w.seg_cnt, cap / racer::kMinStretch + 2, false, stream))) return rc;
  if ((rc = dev_alloc(&w.def_list, cap, false, stream))) return rc;
  if ((rc = dev_alloc(&w.loc, cap, false, stream))) return rc;
  if ((rc = dev_alloc(&w.hents, hsize, true, stream))) return rc;
  if ((rc = dev_alloc(&w.hslot_u, hsize, false, stream))) return rc;
  if ((rc = dev_alloc(&w.heads, hsize, true, stream))) return rc;
  if ((rc = dev_alloc(&w.rec, cap, false, stream))) return rc;
  if ((rc = dev_alloc(&w.u_way, cap, false, stream))) return rc;
  if ((rc = dev_alloc(&w.staging, cap * p->cfg.row_bytes, false, stream))) return rc;
  w.hmask = static_cast<uint32_t>(hsize - 1);
  w.headmask = static_cast<uint32_t>(hsize - 1);
  p->ws_cap = cap;
  return RACER_OK;
}

// The remaining work spaces grow on demand (a growth waits for the streams that may still use the old buffer);
// pool_reserve sizes them all ahead of time.
// fp32 partial outputs of query tiles cut into pieces.  A step asks for more than it needs (want): how many there are follows
// the shape of the batch, and steps that each need a little more than any before them must not each wait and allocate.
int32_t ensure_partials(racer_pool* p, uint64_t need, uint64_t want, hipStream_t stream) {
  if (need <= p->hp_cap) return RACER_OK;
  HIP_TRY(hipStreamSynchronize(p->last_stream));
  HIP_TRY(hipStreamSynchronize(stream));
  if (p->hp_dev) HIP_TRY(hipFree(p->hp_dev));
  p->hp_dev = nullptr;
  p->hp_cap = 0;
  HIP_TRY(hipMalloc(reinterpret_cast<void**>(&p->hp_dev), want));
  p->hp_cap = want;
  p->ws_allocs += 1;
  return RACER_OK;
}

int32_t ensure_lists(racer_pool* p, uint64_t need, uint64_t want) {  // device copy of a step's host-built lists
  if (need <= p->hl_cap) return RACER_OK;
  HIP_TRY(hipStreamSynchronize(p->last_stream));
  if (p->hl_dev) HIP_TRY(hipFree(p->hl_dev));
  p->hl_dev = nullptr;
  p->hl_cap = 0;
  HIP_TRY(hipMalloc(reinterpret_cast<void**>(&p->hl_dev), want));
  p->hl_cap = want;
  p->ws_allocs += 1;
  return RACER_OK;
}

// Activation work space of a step: six matrices (xn, u, q, o and two layer buffers) of `slot` bytes each.
int32_t ensure_hstu_ws(racer_pool* p, uint64_t slot, hipStream_t stream) {
  if (slot <= p->hw_slot) return RACER_OK;
  HIP_TRY(hipStreamSynchronize(stream));
  HIP_TRY(hipStreamSynchronize(p->last_stream));
  if (p->hw_buf) HIP_TRY(hipFree(p->hw_buf));
  p->hw_buf = nullptr;
  p->hw_slot = 0;
  HIP_TRY(hipMalloc(reinterpret_cast<void**>(&p->hw_buf), slot * 6));
  p->hw_slot = slot;
  p->ws_allocs += 1;
  return RACER_OK;
}

// The marks of requests whose timestamps decrease somewhere (the number of the step that found it; 0: none).
int32_t ensure_ts_marks(racer_pool* p, uint64_t B, hipStream_t stream) {
  if (B <= p->ts_marks_cap) return RACER_OK;
  HIP_TRY(hipStreamSynchronize(p->last_stream));
  if (p->ts_marks) HIP_TRY(hipFree(p->ts_marks));
  p->ts_marks = nullptr;
  p->ts_marks_cap = 0;
  const uint64_t cap = std::max<uint64_t>(B, 256);
  int32_t rc = dev_alloc(&p->ts_marks, cap, true, stream);
  if (rc) return rc;
  p->ts_marks_cap = cap;
  p->ws_allocs += 1;
  return RACER_OK;
}

}  // namespace

extern "C" {

const char* racer_last_error(void) { return g_last_error.c_str(); }

int32_t pool_create(void* dev_base, uint64_t bytes, uint64_t page_size, const racer_pool_cfg* cfg, racer_pool_t** out) {
  if (!cfg || !out) return RACER_EINVAL;
  *out = nullptr;
  if (cfg->row_bytes == 0 || cfg->row_bytes % 16 != 0) return RACER_EINVAL;
  if (cfg->elem != RACER_ELEM_F32 && cfg->elem != RACER_ELEM_BF16) return RACER_EINVAL;
  if (cfg->page_tokens == 0 || !is_pow2(cfg->w_max) || cfg->w_max > 32) return RACER_EINVAL;
  if (page_size == 0 || bytes == 0 || bytes % page_size != 0 || page_size % cfg->row_bytes != 0) return RACER_EINVAL;
  const uint64_t n_pages = bytes / page_size;
  if (n_pages % cfg->w_max != 0 || n_pages >= (1ull << 31)) return RACER_EINVAL;
  if (cfg->rows >= 0xFFFFFFFFull) return RACER_EINVAL;
  if (!(cfg->emb_frac0 >= 0.0 && cfg->emb_frac0 <= 1.0)) return RACER_EINVAL;
  const uint64_t spp = page_size / cfg->row_bytes;
  const uint64_t sets = n_pages / cfg->w_max * spp;
  if (spp >= (1ull << 31) || sets >= (1ull << 32)) return RACER_EINVAL;
  if (dev_base && (reinterpret_cast<uintptr_t>(dev_base) & 255)) return RACER_EINVAL;

  racer_pool* p = new (std::nothrow) racer_pool(n_pages, *cfg, static_cast<uint32_t>(spp));
  if (!p) return RACER_ENOMEM;
  p->base = static_cast<uint8_t*>(dev_base);
  p->bytes = bytes;
  p->page_size = page_size;
  p->device = dev_base != nullptr;
  p->host.seed_emb(static_cast<uint64_t>(std::llround(cfg->emb_frac0 * static_cast<double>(n_pages))));
  if (p->device) {
    int32_t rc = RACER_OK;
    const uint64_t n_tags = sets * cfg->w_max;
    if ((rc = dev_alloc(&p->d_tags, n_tags, false, nullptr)) || (rc = dev_alloc(&p->d_stamps, n_tags, true, nullptr)) ||
        (rc = dev_alloc(&p->d_emb_pages, n_pages, true, nullptr)) ||
        (rc = dev_alloc(&p->d_counters, racer::kCtrCount * racer::kCtrShards, true, nullptr))) {
      pool_destroy(p);
      return rc;
    }
    hipError_t e = racer::launch_fill_u32(p->d_tags, n_tags, RACER_TAG_EMPTY, nullptr);
    if (e == hipSuccess && p->host.n_emb())
      e = hipMemcpy(p->d_emb_pages, p->host.emb_pages().data(), p->host.n_emb() * sizeof(int32_t), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e == hipSuccess && cfg->host_table) {
      void* dp = nullptr;
      e = hipHostGetDevicePointer(&dp, const_cast<void*>(cfg->host_table), 0);
      p->d_table = static_cast<const uint8_t*>(dp);
      if (e == hipSuccess) p->tables.push_back(racer::TableDesc{0, cfg->rows, p->d_table, cfg->row_bytes, 0});
    }
    if (e != hipSuccess) {
      pool_destroy(p);
      return hip_fail(e, "pool_create device setup");
    }
  }
  *out = p;
  return RACER_OK;
}

int32_t pool_destroy(racer_pool_t* p) {
  if (!p) return RACER_EINVAL;
  if (p->device) {
    (void)hipStreamSynchronize(p->last_stream);
    free_miss_ws(p);
    p->stage.release();
    p->hstage.release();
    for (const racer_pool::ProfMark& m : p->prof) {
      (void)hipEventDestroy(m.a);
      (void)hipEventDestroy(m.b);
    }
    for (hipEvent_t e : p->prof_spare) (void)hipEventDestroy(e);
    (void)hipFree(p->d_tables);
    (void)hipFree(p->d_tags);
    (void)hipFree(p->d_stamps);
    (void)hipFree(p->d_emb_pages);
    (void)hipFree(p->d_counters);
    (void)hipFree(p->hw_buf);
    (void)hipFree(p->hl_dev);
    (void)hipFree(p->hp_dev);
    (void)hipFree(p->ts_marks);
  }
  delete p;
  return RACER_OK;
}

int32_t pool_set_split(racer_pool_t* p, double emb_frac, void* stream_v, double* achieved) {
  if (!p) return RACER_EINVAL;
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  const uint64_t G = p->host.layer_pages();
  // The host bookkeeping changes first (the device half needs its result); a copy of it is kept until the device
  // half has been queued, and put back if that fails, so that host and device never disagree about the EMB pages.
  std::unique_ptr<racer::HostPool> undo;
  if (p->device) undo.reset(new (std::nothrow) racer::HostPool(p->host));
  if (p->device && !undo) return RACER_ENOMEM;
  const racer::SplitPlan plan = p->host.set_split(emb_frac);
  if (plan.rc < 0) return plan.rc;
  int32_t rc = RACER_OK;
  if (p->device && plan.new_emb != plan.old_emb) {
    rc = [&]() -> int32_t {
      if (fault_injected("split")) return hip_fail(hipErrorUnknown, "pool_set_split (injected fault)");
      if (plan.new_emb > plan.old_emb) {
        // newly mapped logical pages: ship their physical ids; the new ways are already empty
        const uint64_t count = plan.new_emb - plan.old_emb;
        uint8_t* buf;
        int which;
        int32_t r = p->stage.acquire(count * sizeof(int32_t), &buf, &which);
        if (r) return r;
        std::memcpy(buf, p->host.emb_pages().data() + plan.old_emb, count * sizeof(int32_t));
        HIP_TRY(hipMemcpyAsync(p->d_emb_pages + plan.old_emb, buf, count * sizeof(int32_t), hipMemcpyHostToDevice, stream));
        return p->stage.mark(which, stream);
      }
      const uint32_t old_full = static_cast<uint32_t>(plan.old_emb / G);
      const uint32_t old_part = static_cast<uint32_t>((plan.old_emb % G) * p->host.spp());
      HIP_TRY(racer::launch_emb_shrink(p->view(), old_full, old_part, stream));
      return RACER_OK;
    }();
    if (rc) {
      p->host = std::move(*undo);  // nothing has changed: the device still holds the old split's state
      if (achieved) *achieved = static_cast<double>(p->host.n_emb()) / static_cast<double>(p->host.n_pages());
      return rc;
    }
    p->last_stream = stream;
  }
  if (achieved) *achieved = static_cast<double>(p->host.n_emb()) / static_cast<double>(p->host.n_pages());
  return plan.rc;
}

int32_t pool_stats(racer_pool_t* p, racer_pool_stats* out) {
  if (!p || !out) return RACER_EINVAL;
  std::memset(out, 0, sizeof(*out));
  if (p->device) {
    HIP_TRY(hipStreamSynchronize(p->last_stream));
    unsigned long long shards[racer::kCtrShards][racer::kCtrCount];
    HIP_TRY(hipMemcpy(shards, p->d_counters, sizeof(shards), hipMemcpyDeviceToHost));
    unsigned long long c[racer::kCtrCount] = {};
    for (int sh = 0; sh < racer::kCtrShards; ++sh)
      for (int k = 0; k < racer::kCtrCount; ++k) c[k] += shards[sh][k];
    out->lookups = c[racer::kCtrLookups];
    out->hits = c[racer::kCtrHits];
    out->misses = c[racer::kCtrMisses];
    out->unique_misses = c[racer::kCtrUnique];
    out->inserted = c[racer::kCtrInserted];
    out->evicted = c[racer::kCtrEvicted];
    out->bypassed = c[racer::kCtrBypassed];
    out->invalid_ids = c[racer::kCtrInvalid];
    out->shrink_evicted = c[racer::kCtrShrinkEvicted];
    out->shrink_moved = c[racer::kCtrShrinkMoved];
    out->bad_pages = c[racer::kCtrBadPages];
    out->unordered_ts = c[racer::kCtrUnorderedTs];
  }
  out->ws_allocs = p->ws_allocs + p->stage.allocs + p->hstage.allocs;
  out->pages_total = p->host.n_pages();
  out->pages_emb = p->host.n_emb();
  out->pages_kv_free = p->host.free_count();
  out->pages_kv_used = p->host.n_pages() - p->host.n_emb() - p->host.free_count();
  out->seqs_resident = p->host.seqs_resident();
  out->seqs_evicted = p->host.seqs_evicted();
  out->batch = p->batch;
  return RACER_OK;
}

int32_t pool_dump(racer_pool_t* p, int64_t* emb_pages, uint8_t* owner) {
  if (!p) return RACER_EINVAL;
  if (emb_pages)
    for (uint64_t k = 0; k < p->host.n_emb(); ++k) emb_pages[k] = p->host.emb_pages()[k];
  if (owner) std::memcpy(owner, p->host.owner().data(), p->host.n_pages());
  return RACER_OK;
}

int32_t emb_cache_dump(racer_pool_t* p, uint32_t* tags, uint32_t* stamps) {
  if (!p || !p->device) return RACER_EINVAL;
  HIP_TRY(hipStreamSynchronize(p->last_stream));
  const uint64_t bytes = p->host.sets() * p->cfg.w_max * sizeof(uint32_t);
  if (tags) HIP_TRY(hipMemcpy(tags, p->d_tags, bytes, hipMemcpyDeviceToHost));
  if (stamps) HIP_TRY(hipMemcpy(stamps, p->d_stamps, bytes, hipMemcpyDeviceToHost));
  return RACER_OK;
}

uint64_t pool_num_sets(const racer_pool_t* p) { return p ? p->host.sets() : 0; }

int64_t pool_slot_of(const racer_pool_t* p, uint64_t set, uint32_t way) { return p ? p->host.slot_of(set, way) : -1; }

int32_t kv_seq_reserve(racer_pool_t* p, uint64_t key, uint32_t tokens, int32_t* pages_out, uint32_t cap, uint32_t* n_out) {
  return p ? p->host.reserve(key, tokens, pages_out, cap, n_out) : RACER_EINVAL;
}
int32_t kv_seq_lookup(const racer_pool_t* p, uint64_t key, uint32_t* tokens, int32_t* pages_out, uint32_t cap, uint32_t* n_out) {
  return p ? p->host.lookup(key, tokens, pages_out, cap, n_out) : RACER_EINVAL;
}
int32_t kv_seq_pin(racer_pool_t* p, uint64_t key) { return p ? p->host.pin(key) : RACER_EINVAL; }
int32_t kv_seq_unpin(racer_pool_t* p, uint64_t key) { return p ? p->host.unpin(key) : RACER_EINVAL; }
int32_t kv_seq_release(racer_pool_t* p, uint64_t key) { return p ? p->host.release(key) : RACER_EINVAL; }

}  // extern "C"

namespace {

// emb_lookup and emb_lookup_tables: `ids` names the rows, the rest is the same.
int32_t lookup(racer_pool* p, const racer::IdSrc& ids, uint64_t n, uint32_t bag, void* out, uint8_t* hit_flags, hipStream_t stream) {
  if (bag == 0 || bag > 64 || n % bag != 0 || n >= 0xFFFFFFFFull) return RACER_EINVAL;
  if (n && (!ids.ids || !out)) return RACER_EINVAL;
  p->batch += 1;  // one call = one LRU batch, empty or not
  if (n == 0) return RACER_OK;
  int32_t rc = ensure_miss_ws(p, n, stream);
  if (rc) return rc;
  p->last_stream = stream;
  const racer::EmbView v = p->view();
  {
    ProfScope t(p, RACER_PROF_EMB_GATHER, stream);
    HIP_TRY(racer::launch_emb_probe(v, p->ws, ids, static_cast<uint32_t>(n), bag, static_cast<uint8_t*>(out), hit_flags, p->batch, stream));
  }
  ProfScope t(p, RACER_PROF_EMB_MISS, stream);
  HIP_TRY(racer::launch_emb_miss_path(v, p->ws, static_cast<uint32_t>(n), bag, static_cast<uint8_t*>(out), p->batch, stream));
  return RACER_OK;
}

}  // namespace

extern "C" {

int32_t emb_lookup(racer_pool_t* p, const int64_t* ids, uint64_t n, uint32_t bag, void* out, uint8_t* hit_flags, void* stream_v) {
  if (!p || !p->device || !p->d_table) return RACER_EINVAL;
  return lookup(p, racer::IdSrc{ids, nullptr}, n, bag, out, hit_flags, static_cast<hipStream_t>(stream_v));
}

int32_t emb_lookup_noalloc(racer_pool_t* p, const int64_t* ids, uint64_t n, uint32_t bag, void* out, uint8_t* hit_flags,
                           void* stream_v) {
  if (!p || !p->device || !p->d_table) return RACER_EINVAL;
  if (bag == 0 || bag > 64 || n % bag != 0) return RACER_EINVAL;
  if (n && (!ids || !out)) return RACER_EINVAL;
  if (n > kNoallocMaxLookups || n * p->cfg.row_bytes > kNoallocStagingBytes) {
    g_last_error = "emb_lookup_noalloc: batch beyond the fixed work space (RACER_NOALLOC_MAX_LOOKUPS lookups, "
                   "RACER_NOALLOC_MAX_ROW_BYTES_TOTAL bytes of rows)";
    return RACER_ERANGE;
  }
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  uint8_t* base = nullptr;
  int32_t rc = scratch_address(&base);
  if (rc) return rc;
  p->batch += 1;  // one call = one LRU batch, empty or not
  if (n == 0) return RACER_OK;
  uint64_t hsize = 2048;
  while (hsize < 2 * n) hsize <<= 1;  // <= kNoallocHash
  racer::MissWs ws{};
  ws.any = reinterpret_cast<uint32_t*>(base);
  ws.hents = reinterpret_cast<racer::HashEnt*>(base + kOffHents);
  ws.heads = reinterpret_cast<unsigned long long*>(ws.hents + hsize);
  ws.hmask = ws.headmask = static_cast<uint32_t>(hsize - 1);
  ws.seg_cnt = reinterpret_cast<uint32_t*>(base + kOffSegCnt);
  ws.def_list = reinterpret_cast<uint32_t*>(base + kOffDefList);
  ws.loc = reinterpret_cast<int64_t*>(base + kOffLoc);
  ws.hslot_u = reinterpret_cast<uint32_t*>(base + kOffHslot);
  ws.rec = reinterpret_cast<uint4*>(base + kOffRec);
  ws.u_way = reinterpret_cast<int32_t*>(base + kOffWay);
  ws.staging = base + kOffStaging;
  // The array keeps the last call's contents, whichever pool made it: the two tables whose entries are told apart by
  // the batch number must start at zero.  A fill kernel, so that the call can be captured into a graph.
  HIP_TRY(racer::launch_fill_u32(ws.any, (kOffHents + kClearBytes * hsize) / 4, 0u, stream));
  p->last_stream = stream;
  const racer::EmbView v = p->view();
  HIP_TRY(racer::launch_emb_probe(v, ws, racer::IdSrc{ids, nullptr}, static_cast<uint32_t>(n), bag, static_cast<uint8_t*>(out),
                                  hit_flags, p->batch, stream));
  HIP_TRY(racer::launch_emb_miss_path(v, ws, static_cast<uint32_t>(n), bag, static_cast<uint8_t*>(out), p->batch, stream));
  return RACER_OK;
}

int32_t pool_add_table(racer_pool_t* p, const void* host_table, uint64_t rows, uint32_t row_bytes, uint32_t* table_out) {
  if (!p || !p->device || !p->d_table || p->tables.empty() || !host_table) return RACER_EINVAL;
  if (rows == 0 || row_bytes == 0 || row_bytes % 16 != 0 || row_bytes > p->cfg.row_bytes) return RACER_EINVAL;
  if (p->tables.size() >= racer::kMaxTables) return RACER_EINVAL;
  const uint64_t base = p->tables.back().base + p->tables.back().rows;
  if (base + rows >= 0xFFFFFFFFull) return RACER_EINVAL;  // global ids are the 32-bit cache tags
  void* dp = nullptr;
  HIP_TRY(hipHostGetDevicePointer(&dp, const_cast<void*>(host_table), 0));
  // lookups in flight read the old descriptor array: wait for them, then replace it
  HIP_TRY(hipStreamSynchronize(p->last_stream));
  std::vector<racer::TableDesc> next = p->tables;
  next.push_back(racer::TableDesc{base, rows, static_cast<const uint8_t*>(dp), row_bytes, 0});
  racer::TableDesc* d_next = nullptr;
  HIP_TRY(hipMalloc(reinterpret_cast<void**>(&d_next), sizeof(racer::TableDesc) * next.size()));
  hipError_t e = hipMemcpy(d_next, next.data(), sizeof(racer::TableDesc) * next.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipFree(d_next);
    return hip_fail(e, "pool_add_table");
  }
  if (p->d_tables) (void)hipFree(p->d_tables);
  p->d_tables = d_next;
  p->tables.swap(next);
  if (table_out) *table_out = static_cast<uint32_t>(p->tables.size() - 1);
  return RACER_OK;
}

int32_t emb_lookup_tables(racer_pool_t* p, const uint32_t* table_of, const int64_t* ids, uint64_t n, uint32_t bag,
                          void* out, uint8_t* hit_flags, void* stream_v) {
  if (!p || !p->device || !p->d_table) return RACER_EINVAL;
  if (n >= 0xFFFFFFFFull || (n && (!table_of || !ids))) return RACER_EINVAL;
  if (p->tables.size() < 2) return RACER_EINVAL;  // one table: emb_lookup
  return lookup(p, racer::IdSrc{ids, table_of}, n, bag, out, hit_flags, static_cast<hipStream_t>(stream_v));
}

int32_t emb_refill(racer_pool_t* p, const int64_t* ids, uint64_t n, void* stream_v) {
  if (!p || !p->device || !p->d_table) return RACER_EINVAL;
  if (n >= 0xFFFFFFFFull || (n && !ids)) return RACER_EINVAL;
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  p->batch += 1;  // a batch of its own in LRU time (and a fresh key for the dedupe table)
  if (n == 0) return RACER_OK;
  int32_t rc = ensure_miss_ws(p, n, stream);
  if (rc) return rc;
  p->last_stream = stream;
  ProfScope t(p, RACER_PROF_EMB_MISS, stream);
  HIP_TRY(racer::launch_emb_refill(p->view(), p->ws, racer::IdSrc{ids, nullptr}, static_cast<uint32_t>(n), p->batch, stream));
  return RACER_OK;
}

// ---- HSTU ---------------------------------------------------------------------------------

int32_t hstu_model_create(const racer_hstu_cfg* cfg, const racer_hstu_weights* w, racer_hstu_t** out) {
  if (!cfg || !w || !out) return RACER_EINVAL;
  *out = nullptr;
  if (cfg->L == 0 || cfg->H == 0 || cfg->d == 0 || cfg->d % cfg->H != 0) return RACER_EINVAL;
  if (cfg->page_tokens == 0 || cfg->n_pos == 0 || cfg->n_time == 0 || cfg->n_time > 64) return RACER_EINVAL;
  constexpr uint32_t kMaxWidth = 1024;
  static_assert(kMaxWidth / 64 <= racer::kMaxHeads, "a list entry of the bf16 attention has four bits for the head");
  if (!(cfg->n_scale > 0.0f) || !(cfg->eps > 0.0f) || cfg->d > kMaxWidth) return RACER_EINVAL;
  const uint32_t dh = cfg->d / cfg->H;
  if (cfg->elem == RACER_ELEM_BF16) {
    if (dh != 64 || cfg->d % 64 != 0 || cfg->page_tokens % 8 != 0) return RACER_EINVAL;
  } else if (cfg->elem == RACER_ELEM_F32) {
    if (dh > 64 || cfg->d % 16 != 0) return RACER_EINVAL;
  } else {
    return RACER_EINVAL;
  }
  const void* ptrs[] = {w->ln1_g, w->ln1_b, w->w1, w->b1, w->ln2_g, w->ln2_b, w->w2, w->b2, w->pos, w->time};
  for (const void* q : ptrs)
    if (!q) return RACER_EINVAL;
  racer_hstu* m = new (std::nothrow) racer_hstu();
  if (!m) return RACER_ENOMEM;
  m->cfg = *cfg;
  m->w = *w;
  if (cfg->elem == RACER_ELEM_BF16) {
    const uint64_t d = cfg->d;
    const bool fused = racer::layer_halves_fused(racer::HstuDims{cfg->L, cfg->d, cfg->H, cfg->d / cfg->H, cfg->elem});
    hipError_t e = hipMalloc(&m->w1t, cfg->L * d * 4 * d * 2);
    if (e == hipSuccess) e = hipMalloc(&m->w2t, cfg->L * d * d * 2);
    for (uint32_t l = 0; l < cfg->L && e == hipSuccess; ++l) {
      e = racer::launch_weight_copy(static_cast<const uint16_t*>(w->w1) + l * d * 4 * d,
                                          static_cast<uint16_t*>(m->w1t) + l * d * 4 * d, cfg->d, 4 * cfg->d, fused, nullptr);
      if (e == hipSuccess)
        e = racer::launch_weight_copy(static_cast<const uint16_t*>(w->w2) + l * d * d,
                                            static_cast<uint16_t*>(m->w2t) + l * d * d, cfg->d, cfg->d, fused, nullptr);
    }
    const uint64_t n_pos_all = static_cast<uint64_t>(cfg->L) * cfg->H * cfg->n_pos;
    const uint64_t n_time_all = static_cast<uint64_t>(cfg->L) * cfg->H * cfg->n_time;
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&m->pos_s), n_pos_all * sizeof(float));
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&m->time_s), n_time_all * sizeof(float));
    if (e == hipSuccess) e = racer::launch_scale_bias(static_cast<const float*>(w->pos), m->pos_s, n_pos_all, nullptr);
    if (e == hipSuccess) e = racer::launch_scale_bias(static_cast<const float*>(w->time), m->time_s, n_time_all, nullptr);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
      hstu_model_destroy(m);
      return hip_fail(e, "hstu_model_create weight preparation");
    }
  }
  *out = m;
  return RACER_OK;
}

int32_t hstu_model_destroy(racer_hstu_t* m) {
  if (!m) return RACER_EINVAL;
  (void)hipFree(m->w1t);
  (void)hipFree(m->w2t);
  (void)hipFree(m->pos_s);
  (void)hipFree(m->time_s);
  delete m;
  return RACER_OK;
}

}  // extern "C"

namespace {

// Upper bounds of a step's list bytes and partial-output bytes for up to B requests, N new tokens and sequences of up
// to max_seq tokens (pool_reserve sizes the work spaces with them; prepare_step's own sizes never exceed them).
struct StepBounds { uint64_t list_bytes, partial_bytes; };
StepBounds step_bounds(uint64_t B, uint64_t N, uint64_t max_seq, uint32_t H, uint32_t page_tokens) {
  const racer::AttnBounds a = racer::attn_bounds(B, N, max_seq, H, page_tokens);
  StepBounds b;
  b.list_bytes = sizeof(racer::ReqDev) * (B + 1) + 4 * (N / 32 + B + 2) + sizeof(racer::F32Tile) * (N / racer::kF32Queries + B) +
                 (sizeof(racer::AttnItem) + sizeof(uint32_t)) * a.items + sizeof(racer::AttnWork) * a.work +
                 sizeof(racer::RowTile) * (a.items + 1) + 8 * 256;
  b.partial_bytes = a.work * 128 * 64 * sizeof(float);
  return b;
}

struct StepCtx {
  racer::HstuDims hd;
  racer::KvView kv;
  racer::StepLists sl;
  uint64_t esize;
  bool fused;   // layer halves in one kernel each
  bool joined;  // a back half and the next front half in one kernel
  bool begins;  // the first front half's kernel begins the step, with:
  racer::ListArg arg;
  uint64_t list_bytes;
};

// Validate the requests, build the attention work lists and the row -> request maps, ship them to the device on
// `stream`, and have the timestamps looked at (or, if the caller says that it can, leave these two to the first layer's kernel).
int32_t prepare_step(racer_pool* p, racer_hstu* m, const racer_hstu_req* reqs, uint32_t B, uint64_t n_page_entries,
                     const int64_t* ts, hipStream_t stream, bool can_begin, StepCtx* ctx) {
  const racer_hstu_cfg& c = m->cfg;
  if (!p->device || c.page_tokens != p->cfg.page_tokens || c.elem != p->cfg.elem) return RACER_EINVAL;
  const uint64_t esize = c.elem == RACER_ELEM_BF16 ? 2 : 4;
  if (static_cast<uint64_t>(c.page_tokens) * 2 * c.L * c.d * esize != p->page_size) return RACER_EINVAL;
  uint64_t N = 0, cached = 0;
  uint32_t longest = 0;
  for (uint32_t r = 0; r < B; ++r) {
    const racer_hstu_req& q = reqs[r];
    const uint64_t S = static_cast<uint64_t>(q.prefix_len) + q.new_len;
    const uint64_t need = (S + c.page_tokens - 1) / c.page_tokens;
    if (q.page_table_off + need > n_page_entries) return RACER_EINVAL;
    if (q.x_off != N) return RACER_EINVAL;  // rows are packed request after request
    if (q.page_table_off >= (1ull << 32) || q.ts_off >= (1ull << 32) || S >= (1ull << 31)) return RACER_EINVAL;
    N += q.new_len;
    cached += q.prefix_len;
    longest = std::max(longest, static_cast<uint32_t>(S));
  }
  if (N >= (1ull << 31) || B >= (1u << 24)) return RACER_EINVAL;
  const bool fp32 = c.elem != RACER_ELEM_BF16;
  ctx->esize = esize;
  uint32_t pt_shift = 32;
  for (uint32_t b = 0; b < 32; ++b)
    if ((1u << b) == c.page_tokens) pt_shift = b;
  ctx->hd = racer::HstuDims{c.L, c.d, c.H, c.d / c.H, c.elem, c.page_tokens, c.n_pos, c.n_time, 1.0f / c.n_scale, c.eps, pt_shift};
  ctx->kv = racer::KvView{p->base, p->page_size, static_cast<uint32_t>(p->host.n_pages()), p->d_counters};
  ctx->fused = racer::layer_halves_fused(ctx->hd);
  racer::StepLists& sl = ctx->sl;
  sl = racer::StepLists{};
  sl.B = B;
  sl.N = static_cast<uint32_t>(N);
  ctx->joined = racer::layers_joined(ctx->hd, sl.N, B, cached);
  if (N == 0) return RACER_OK;

  StepScratch& w = p->step;
  w.row_tiles.clear();
  w.f32_tiles.clear();
  w.reqs.resize(B);
  for (uint32_t r = 0; r < B; ++r)
    w.reqs[r] = racer::ReqDev{reqs[r].prefix_len, reqs[r].new_len, static_cast<uint32_t>(reqs[r].page_table_off),
                              static_cast<uint32_t>(reqs[r].ts_off), static_cast<uint32_t>(reqs[r].x_off)};
  w.attn.build(w.reqs.data(), fp32 ? 0 : B, c.H, c.page_tokens);
  if (fp32)
    for (uint32_t r = 0; r < B; ++r)
      for (uint32_t q0 = 0; q0 < reqs[r].new_len; q0 += racer::kF32Queries) {
        w.f32_tiles.push_back({r, q0});
        sl.f32_keys += reqs[r].prefix_len + std::min(q0 + racer::kF32Queries, reqs[r].new_len);
      }
  const uint64_t partial_bytes = static_cast<uint64_t>(w.attn.n_slots) * 128 * 64 * sizeof(float);
  int32_t rc = ensure_partials(p, partial_bytes, partial_bytes + partial_bytes / 4, stream);
  if (rc) return rc;
  if (!fp32 && !ctx->fused)
    for (uint32_t r = 0; r < B; ++r)
      for (uint32_t t0 = 0; t0 < reqs[r].new_len; t0 += 128)
        w.row_tiles.push_back({static_cast<uint32_t>(reqs[r].x_off) + t0, std::min<uint32_t>(128, reqs[r].new_len - t0), r, 0});

  // one block of memory for all lists
  const uint64_t n_groups32 = ctx->fused ? (N + 31) / 32 + 1 : 0;
  uint64_t total = 0;
  auto place = [&](uint64_t bytes) {
    const uint64_t at = total;
    total = (total + bytes + 15) & ~15ull;
    return at;
  };
  const uint64_t off_reqs = place(sizeof(racer::ReqDev) * B);
  const uint64_t off_items = place(sizeof(racer::AttnItem) * w.attn.items.size());
  const uint64_t off_work = place(sizeof(racer::AttnWork) * w.attn.work.size());
  const uint64_t off_groups = place(sizeof(uint32_t) * w.attn.groups.size());
  const uint64_t off_row_tiles = place(sizeof(racer::RowTile) * w.row_tiles.size());
  const uint64_t off_group_req = place(sizeof(uint32_t) * n_groups32);  // request of every 32nd row, and of the last one
  const uint64_t off_f32_tiles = place(sizeof(racer::F32Tile) * w.f32_tiles.size());
  if ((rc = ensure_lists(p, total, total * 2)) || (rc = ensure_ts_marks(p, B, stream))) return rc;
  p->step_epoch += 1;
  // Small lists travel as an argument of the kernel that begins the step, larger ones it reads from pinned staging.
  const bool by_argument = total <= racer::kListArgBytes;
  uint8_t* hbuf = ctx->arg.bytes;
  int which = 0;
  if (!by_argument && (rc = p->hstage.acquire(total, &hbuf, &which))) return rc;
  auto put = [&](uint64_t at, const auto& v) {
    if (!v.empty()) std::memcpy(hbuf + at, v.data(), v.size() * sizeof(v[0]));
  };
  put(off_reqs, w.reqs);
  put(off_items, w.attn.items);
  put(off_work, w.attn.work);
  put(off_groups, w.attn.groups);
  put(off_row_tiles, w.row_tiles);
  put(off_f32_tiles, w.f32_tiles);
  if (ctx->fused) {
    uint32_t* gr = reinterpret_cast<uint32_t*>(hbuf + off_group_req);
    uint64_t next = 0;
    uint32_t last = 0;
    for (uint32_t r = 0; r < B; ++r) {
      const uint64_t end = reqs[r].x_off + reqs[r].new_len;
      if (reqs[r].new_len) last = r;
      for (; next < end; next += 32) *gr++ = r;
    }
    *gr = last;
  }

  sl.reqs = reinterpret_cast<const racer::ReqDev*>(p->hl_dev + off_reqs);
  sl.ts_marks = p->ts_marks;
  sl.epoch = p->step_epoch;
  sl.items = reinterpret_cast<const racer::AttnItem*>(p->hl_dev + off_items);
  sl.work = reinterpret_cast<const racer::AttnWork*>(p->hl_dev + off_work);
  std::copy(std::begin(w.attn.begin), std::end(w.attn.begin), sl.dies.begin);
  sl.dies.piece = w.attn.piece;
  sl.n_blocks = w.attn.blocks;
  sl.turns = w.attn.turns;
  sl.groups = reinterpret_cast<const uint32_t*>(p->hl_dev + off_groups);
  sl.n_groups = static_cast<uint32_t>(w.attn.groups.size());
  uint64_t row_blocks = 0;  // of four rows, of all cut query tiles
  for (uint32_t i : w.attn.groups) row_blocks += (std::min<uint32_t>(128, w.attn.items[i].new_len - w.attn.items[i].qt * 128) + 3) / 4;
  sl.sum_rows = racer::sums_by_rows(row_blocks * c.H, w.attn.n_slots, w.attn.groups.size() * c.H);
  sl.partials = reinterpret_cast<float*>(p->hp_dev);
  sl.row_tiles = reinterpret_cast<const racer::RowTile*>(p->hl_dev + off_row_tiles);
  sl.n_row_tiles = static_cast<uint32_t>(w.row_tiles.size());
  sl.group_req = reinterpret_cast<const uint32_t*>(p->hl_dev + off_group_req);
  sl.f32_tiles = reinterpret_cast<const racer::F32Tile*>(p->hl_dev + off_f32_tiles);
  sl.n_f32_tiles = static_cast<uint32_t>(w.f32_tiles.size());
  sl.longest = longest;
  // the lists to the device, and which requests' timestamps never decrease (the attention kernels' 32-bit time paths rely on it)
  ctx->begins = can_begin && by_argument && ctx->joined && racer::begin_joins(sl, longest);
  ctx->list_bytes = total;
  if (ctx->begins) return RACER_OK;
  HIP_TRY(racer::launch_begin_step(sl, longest, ts, p->d_counters, by_argument ? &ctx->arg : nullptr, hbuf, p->hl_dev, total, stream));
  if (!by_argument && (rc = p->hstage.mark(which, stream))) return rc;
  return RACER_OK;
}

}  // namespace

extern "C" {

int32_t pool_reserve(racer_pool_t* p, const racer_hstu_t* m, const racer_reserve* r, void* stream_v) {
  if (!p || !r || !p->device) return RACER_EINVAL;
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  int32_t rc;
  if ((rc = p->stage.reserve(p->host.n_pages() * sizeof(int32_t)))) return rc;  // the largest growth a split change can ship
  if (r->max_lookups) {
    if (r->max_lookups >= 0xFFFFFFFFull) return RACER_EINVAL;
    if ((rc = ensure_miss_ws(p, r->max_lookups, stream))) return rc;
  }
  if (m && r->max_requests) {
    const racer_hstu_cfg& c = m->cfg;
    if (r->max_new_tokens >= (1ull << 31) || r->max_seq_tokens == 0) return RACER_EINVAL;
    const uint64_t esize = c.elem == RACER_ELEM_BF16 ? 2 : 4;
    const StepBounds b = step_bounds(r->max_requests, r->max_new_tokens, r->max_seq_tokens, c.H, c.page_tokens);
    if ((rc = ensure_lists(p, b.list_bytes, b.list_bytes)) || (rc = ensure_ts_marks(p, r->max_requests, stream))) return rc;
    if ((rc = p->hstage.reserve(b.list_bytes))) return rc;
    if (c.elem == RACER_ELEM_BF16)
      p->step.attn.reserve(racer::attn_bounds(r->max_requests, r->max_new_tokens, r->max_seq_tokens, c.H, c.page_tokens), c.H);
    if (c.elem == RACER_ELEM_BF16 && (rc = ensure_partials(p, b.partial_bytes, b.partial_bytes, stream))) return rc;
    if ((rc = ensure_hstu_ws(p, (r->max_new_tokens * c.d * esize + 255) & ~255ull, stream))) return rc;
  }
  return RACER_OK;
}

int32_t hstu_step(racer_pool_t* p, racer_hstu_t* m, const racer_hstu_req* reqs, uint32_t B, const int32_t* page_tables,
                  uint64_t n_page_entries, const void* x_in, const int64_t* ts, void* out, void* stream_v) {
  if (!p || !m || (B && !reqs)) return RACER_EINVAL;
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  const racer_hstu_cfg& c = m->cfg;
  StepCtx ctx;
  int32_t rc = prepare_step(p, m, reqs, B, n_page_entries, ts, stream, /*can_begin=*/true, &ctx);
  if (rc) return rc;
  p->last_stream = stream;
  const racer::StepLists& sl = ctx.sl;
  const uint32_t N = sl.N;
  if (N == 0) return RACER_OK;
  if (!page_tables || !x_in || !ts || !out) return RACER_EINVAL;
  const uint64_t d = c.d;
  if ((rc = ensure_hstu_ws(p, (static_cast<uint64_t>(N) * d * ctx.esize + 255) & ~255ull, stream))) return rc;
  const uint64_t stride = p->hw_slot;
  uint8_t* xn = p->hw_buf;
  uint8_t* u = xn + stride;
  uint8_t* q = u + stride;
  uint8_t* o = q + stride;
  uint8_t* xb[2] = {o + stride, o + 2 * stride};
  const bool bf16 = c.elem == RACER_ELEM_BF16;
  const uint64_t w1_layer = d * 4 * d * ctx.esize, w2_layer = d * d * ctx.esize;
  const void* x_cur = x_in;
  if (ctx.joined) {
    auto f = [](const void* v, uint64_t at) { return static_cast<const float*>(v) + at; };
    auto b8 = [](const void* v) { return static_cast<const uint8_t*>(v); };
    uint8_t* us[2] = {u, xn};  // a layer's back half reads its U while the next one's is written
    auto front = [&](uint32_t l) {
      return racer::LayerFront{l, f(m->w.ln1_g, l * d), f(m->w.ln1_b, l * d), b8(m->w1t) + l * w1_layer, f(m->w.b1, l * 4 * d), us[l & 1], q};
    };
    {
      const racer::LayerFront fr = front(0);
      const racer::BeginStep begin{&ctx.arg, sl.longest, ts, p->d_counters, p->hl_dev, ctx.list_bytes};
      ProfScope t(p, RACER_PROF_GEMM_FRONT, stream);
      HIP_TRY(racer::launch_layer_join(ctx.hd, nullptr, &fr, x_in, ctx.kv, sl, page_tables, stream, ctx.begins ? &begin : nullptr));
    }
    for (uint32_t l = 0; l < c.L; ++l) {
      {
        ProfScope t(p, RACER_PROF_ATTENTION, stream);
        HIP_TRY(racer::launch_attention(ctx.hd, l, q, m->pos_s, m->time_s, ctx.kv, sl, page_tables, ts, o, /*o_half=*/true, stream));
      }
      if (sl.n_groups) {
        ProfScope t(p, RACER_PROF_ATTN_REDUCE, stream);
        HIP_TRY(racer::launch_attention_reduce(ctx.hd, sl, o, /*o_half=*/true, stream));
      }
      const bool last = l + 1 == c.L;
      void* x_next = last ? out : static_cast<void*>(xb[l & 1]);
      const racer::LayerBack bk{o, us[l & 1], f(m->w.ln2_g, l * d), f(m->w.ln2_b, l * d), b8(m->w2t) + l * w2_layer, f(m->w.b2, l * d), x_next};
      racer::LayerFront fr{};
      if (!last) fr = front(l + 1);
      ProfScope t(p, RACER_PROF_GEMM_BACK, stream);
      HIP_TRY(racer::launch_layer_join(ctx.hd, &bk, last ? nullptr : &fr, x_cur, ctx.kv, sl, page_tables, stream));
      x_cur = x_next;
    }
    return RACER_OK;
  }
  for (uint32_t l = 0; l < c.L; ++l) {
    void* x_next = (l + 1 == c.L) ? out : static_cast<void*>(xb[l & 1]);
    const float* ln1_g = static_cast<const float*>(m->w.ln1_g) + l * d;
    const float* ln1_b = static_cast<const float*>(m->w.ln1_b) + l * d;
    const float* ln2_g = static_cast<const float*>(m->w.ln2_g) + l * d;
    const float* ln2_b = static_cast<const float*>(m->w.ln2_b) + l * d;
    const float* b1 = static_cast<const float*>(m->w.b1) + l * 4 * d;
    const float* b2 = static_cast<const float*>(m->w.b2) + l * d;
    const uint8_t* w1 = static_cast<const uint8_t*>(bf16 ? m->w1t : m->w.w1) + l * w1_layer;
    const uint8_t* w2 = static_cast<const uint8_t*>(bf16 ? m->w2t : m->w.w2) + l * w2_layer;
    if (!bf16) {
      auto f = [](const void* v) { return static_cast<const float*>(v); };
      auto fw = [](void* v) { return static_cast<float*>(v); };
      {
        ProfScope t(p, RACER_PROF_GEMM_FRONT, stream);
        HIP_TRY(racer::launch_layer_half_f32(ctx.hd, l, true, f(x_cur), nullptr, ln1_g, ln1_b, f(w1), b1, fw(u), fw(q), ctx.kv, sl,
                                             page_tables, nullptr, nullptr, stream));
      }
      {
        ProfScope t(p, RACER_PROF_ATTENTION, stream);
        HIP_TRY(racer::launch_attention_f32(ctx.hd, l, f(q), f(m->w.pos), f(m->w.time), ctx.kv, sl, page_tables, ts, fw(o), stream));
      }
      ProfScope t(p, RACER_PROF_GEMM_BACK, stream);
      HIP_TRY(racer::launch_layer_half_f32(ctx.hd, l, false, f(o), f(u), ln2_g, ln2_b, f(w2), b2, nullptr, nullptr, ctx.kv, sl, page_tables,
                                           f(x_cur), fw(x_next), stream));
      x_cur = x_next;
      continue;
    }
    if (ctx.fused) {
      ProfScope t(p, RACER_PROF_GEMM_FRONT, stream);
      HIP_TRY(racer::launch_layer_front_fused(ctx.hd, l, x_cur, ln1_g, ln1_b, w1, b1, u, q, ctx.kv, sl, page_tables, stream));
    } else {
      {
        ProfScope t(p, RACER_PROF_LAYERNORM, stream);
        HIP_TRY(racer::launch_layernorm(ctx.hd, x_cur, ln1_g, ln1_b, nullptr, xn, N, stream));
      }
      ProfScope t(p, RACER_PROF_GEMM_FRONT, stream);
      HIP_TRY(racer::launch_gemm_front(ctx.hd, l, xn, w1, b1, u, q, ctx.kv, sl, page_tables, stream));
    }
    {
      ProfScope t(p, RACER_PROF_ATTENTION, stream);
      HIP_TRY(racer::launch_attention(ctx.hd, l, q, m->pos_s, m->time_s, ctx.kv, sl, page_tables, ts, o, /*o_half=*/true, stream));
    }
    if (sl.n_groups) {
      ProfScope t(p, RACER_PROF_ATTN_REDUCE, stream);
      HIP_TRY(racer::launch_attention_reduce(ctx.hd, sl, o, /*o_half=*/true, stream));
    }
    if (ctx.fused) {
      ProfScope t(p, RACER_PROF_GEMM_BACK, stream);
      HIP_TRY(racer::launch_layer_back_fused(ctx.hd, o, u, ln2_g, ln2_b, w2, b2, x_cur, x_next, sl, stream));
    } else {
      {
        ProfScope t(p, RACER_PROF_LAYERNORM, stream);
        HIP_TRY(racer::launch_layernorm(ctx.hd, o, ln2_g, ln2_b, u, xn, N, stream));
      }
      ProfScope t(p, RACER_PROF_GEMM_BACK, stream);
      HIP_TRY(racer::launch_gemm_back(ctx.hd, xn, w2, b2, x_cur, x_next, N, stream));
    }
    x_cur = x_next;
  }
  return RACER_OK;
}

int32_t hstu_attn_paged(racer_pool_t* p, racer_hstu_t* m, uint32_t layer, const racer_hstu_req* reqs, uint32_t B,
                        const int32_t* page_tables, uint64_t n_page_entries, const void* q, const int64_t* ts, void* o,
                        void* stream_v) {
  if (!p || !m || (B && !reqs) || layer >= m->cfg.L) return RACER_EINVAL;
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  StepCtx ctx;
  int32_t rc = prepare_step(p, m, reqs, B, n_page_entries, ts, stream, /*can_begin=*/false, &ctx);
  if (rc) return rc;
  p->last_stream = stream;
  if (ctx.sl.N == 0) return RACER_OK;
  if (!page_tables || !q || !ts || !o) return RACER_EINVAL;
  if (m->cfg.elem == RACER_ELEM_BF16) {
    // the MFMA kernel takes q * log2(e); hstu_step's projection writes it that way, here it is a pre-pass
    if ((rc = ensure_hstu_ws(p, (static_cast<uint64_t>(ctx.sl.N) * m->cfg.d * ctx.esize + 255) & ~255ull, stream))) return rc;
    const uint64_t stride = p->hw_slot;
    void* qs = p->hw_buf + 2 * stride;
    HIP_TRY(racer::launch_scale_q(q, qs, static_cast<uint64_t>(ctx.sl.N) * m->cfg.d, stream));
    q = qs;
  }
  {
    ProfScope t(p, RACER_PROF_ATTENTION, stream);
    if (m->cfg.elem == RACER_ELEM_BF16)
      HIP_TRY(racer::launch_attention(ctx.hd, layer, q, m->pos_s, m->time_s, ctx.kv, ctx.sl, page_tables, ts, o, /*o_half=*/false, stream));
    else
      HIP_TRY(racer::launch_attention_f32(ctx.hd, layer, static_cast<const float*>(q), static_cast<const float*>(m->w.pos),
                                          static_cast<const float*>(m->w.time), ctx.kv, ctx.sl, page_tables, ts, static_cast<float*>(o), stream));
  }
  if (ctx.sl.n_groups) {
    ProfScope t(p, RACER_PROF_ATTN_REDUCE, stream);
    HIP_TRY(racer::launch_attention_reduce(ctx.hd, ctx.sl, o, /*o_half=*/false, stream));
  }
  return RACER_OK;
}

// ---- split controller (host only) --------------------------------------------------------------------------

int32_t alpha_ctl_create(double slo_ms, racer_alpha_ctl_t** out) {
  if (!out) return RACER_EINVAL;
  *out = nullptr;
  if (!(slo_ms > 0.0)) return RACER_EINVAL;
  racer::AlphaController* c = new (std::nothrow) racer::AlphaController(slo_ms);
  if (!c) return RACER_ENOMEM;
  *out = reinterpret_cast<racer_alpha_ctl_t*>(c);
  return RACER_OK;
}

int32_t alpha_ctl_destroy(racer_alpha_ctl_t* ctl) {
  if (!ctl) return RACER_EINVAL;
  delete reinterpret_cast<racer::AlphaController*>(ctl);
  return RACER_OK;
}

int32_t alpha_ctl_decide(racer_alpha_ctl_t* ctl, const racer_alpha_state* s, double* step, double* alpha_next, int32_t* burst) {
  if (!ctl || !s || !alpha_next) return RACER_EINVAL;
  if (!(s->alpha >= 0.0 && s->alpha <= 1.0) || !(s->p99_latency_ms >= 0.0)) return RACER_EINVAL;
  const racer::AlphaState st{s->hot_user_ratio, s->kv_hit_rate, s->emb_hit_rate, s->mean_seq_len, s->slo_violation,
                             s->alpha, s->p99_latency_ms};
  *alpha_next = reinterpret_cast<racer::AlphaController*>(ctl)->decide(st, step, burst);
  return RACER_OK;
}

double alpha_ctl_reward(double slo_satisfaction, double p99_latency_ms, double slo_ms) {
  return racer::alpha_reward(slo_satisfaction, p99_latency_ms, slo_ms);
}

int32_t racer_hbm_probe(const void* dev_base, uint64_t bytes, uint32_t row_bytes, uint64_t n_reads, void* dev_out,
                        uint64_t seed, void* stream_v) {
  if (!dev_base || n_reads == 0 || (row_bytes != 128 && row_bytes != 256 && row_bytes != 512 && row_bytes != 1024)) return RACER_EINVAL;
  if (bytes < row_bytes || (reinterpret_cast<uintptr_t>(dev_base) & 15) || (reinterpret_cast<uintptr_t>(dev_out) & 15)) return RACER_EINVAL;
  HIP_TRY(racer::launch_random_row_reads(dev_base, bytes / row_bytes, row_bytes, n_reads, dev_out, seed,
                                         static_cast<hipStream_t>(stream_v)));
  return RACER_OK;
}

int32_t racer_prof_enable(racer_pool_t* p, int32_t on) {
  if (!p || !p->device) return RACER_EINVAL;
  p->prof_on = on != 0;
  return RACER_OK;
}

int32_t racer_prof_read(racer_pool_t* p, racer_prof* out) {
  if (!p || !p->device || !out) return RACER_EINVAL;
  std::memset(out, 0, sizeof(*out));
  HIP_TRY(hipStreamSynchronize(p->last_stream));
  for (const racer_pool::ProfMark& m : p->prof) {
    float ms = 0.0f;
    HIP_TRY(hipEventElapsedTime(&ms, m.a, m.b));
    out->ms[m.kind] += ms;
    out->launches[m.kind] += 1;
    p->prof_spare.push_back(m.a);
    p->prof_spare.push_back(m.b);
  }
  p->prof.clear();
  return RACER_OK;
}

}  // extern "C"
