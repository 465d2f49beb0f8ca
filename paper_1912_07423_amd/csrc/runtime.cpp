// runtime.cpp -- host runtime behind the C ABI of include/snn.h: validation, derived
// constants, device allocation, on-device network construction, the window schedule
// of the step pipeline, HIP graph replay, profiling and state/raster readback.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <map>
#include <mutex>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <exception>
#include <new>
#include <numeric>
#include <string>
#include <vector>

#include "raster_units.h"
#include "snn_internal.h"

namespace {

thread_local std::string g_error;

struct Failure {
  snn_status code;
  std::string msg;
};

[[noreturn]] void fail(snn_status code, const std::string &msg) { throw Failure{code, msg}; }

void check(hipError_t e, const char *what) {
  if (e != hipSuccess) fail(SNN_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

void refuse_member(const snn_network *net) {
  if (net->owner) fail(SNN_E_STATE, "this network belongs to a batch: advance it with snn_batch_run");
}

template <typename F>
snn_status guarded(F &&f) {
  try {
    f();
    return SNN_OK;
  } catch (const Failure &x) {
    g_error = x.msg;
    return x.code;
  } catch (const std::bad_alloc &) {
    g_error = "host allocation failed";
    return SNN_E_OOM;
  } catch (const std::exception &x) {
    g_error = x.what();
    return SNN_E_INVALID;
  }
}

// ---- device memory --------------------------------------------------------------
// Without an allocator callback, device memory comes from the library's own cache
// (Sec. IV: memory is allocated only when necessary, with hysteresis, so back-to-back
// experiments pay for allocation once).  A freed block is kept per device; a request is
// served by the smallest kept block that is at least as large and at most twice as
// large (plus 1 MiB), else by hipMalloc.  When hipMalloc fails, the device's kept blocks
// are returned to HIP and the request is tried once more.  Blocks are handed back only
// after their network's stream has drained (every caller frees after a stream sync), so
// no work can still touch a reused block.
struct PoolBlock {
  int device;
  void *p;
  size_t bytes;
};
std::mutex g_pool_mutex;
std::vector<PoolBlock> g_pool;  // kept blocks
struct PoolStats {
  uint64_t hits = 0, misses = 0;
};
std::map<int, PoolStats> g_pool_stats;

// Returns the kept blocks of `device` (every device if negative) to HIP.
void pool_release(int device) {
  std::vector<PoolBlock> drop;
  {
    std::lock_guard<std::mutex> lock(g_pool_mutex);
    std::vector<PoolBlock> keep;
    for (const PoolBlock &b : g_pool) (device < 0 || b.device == device ? drop : keep).push_back(b);
    g_pool.swap(keep);
  }
  int cur = 0;
  if (hipGetDevice(&cur) != hipSuccess) return;
  for (const PoolBlock &b : drop) {
    if (b.device != cur) (void)hipSetDevice(b.device);
    (void)hipFree(b.p);
    if (b.device != cur) (void)hipSetDevice(cur);
  }
}

// Serves `bytes` on `device`; *got receives the size of the block handed out (a kept
// block may be up to twice the request plus 1 MiB), which the caller records and hands
// back to pool_free, so a reused block keeps its true size.
void *pool_alloc(int device, size_t bytes, size_t *got) {
  *got = bytes;
  {
    std::lock_guard<std::mutex> lock(g_pool_mutex);
    size_t best = g_pool.size();
    for (size_t k = 0; k < g_pool.size(); ++k) {
      const PoolBlock &b = g_pool[k];
      if (b.device != device || b.bytes < bytes || b.bytes > 2 * bytes + (1u << 20)) continue;
      if (best == g_pool.size() || b.bytes < g_pool[best].bytes) best = k;
    }
    if (best != g_pool.size()) {
      void *p = g_pool[best].p;
      *got = g_pool[best].bytes;
      g_pool.erase(g_pool.begin() + (std::ptrdiff_t)best);
      ++g_pool_stats[device].hits;
      return p;
    }
    ++g_pool_stats[device].misses;
  }
  void *p = nullptr;
  if (hipMalloc(&p, bytes) == hipSuccess) return p;
  (void)hipGetLastError();
  pool_release(device);
  if (hipMalloc(&p, bytes) == hipSuccess) return p;
  (void)hipGetLastError();
  return nullptr;
}

// Keeps a block for reuse; `bytes` is its true size (as pool_alloc reported it).
void pool_free(int device, void *p, size_t bytes) {
  std::lock_guard<std::mutex> lock(g_pool_mutex);
  g_pool.push_back({device, p, bytes});
}

// ---- pinned host staging ------------------------------------------------------------
// Blocks of pinned host memory that kernels write results into.  A call takes one for
// itself and hands it back after its stream has drained, so a block never has two users,
// whatever the threads and streams.  At most kStageKeep free blocks are kept (pinning takes
// longer than the download it serves); snn_memory_cache_release returns them.
constexpr size_t kStageMinBytes = 1u << 20, kStageMaxBytes = 32u << 20;
constexpr size_t kStageKeep = 4;
struct StageBlock {
  void *p = nullptr;
  size_t bytes = 0;
};
std::mutex g_stage_mutex;
std::vector<StageBlock> g_stage;  // free blocks

void stage_release() {
  std::vector<StageBlock> drop;
  {
    std::lock_guard<std::mutex> lock(g_stage_mutex);
    drop.swap(g_stage);
  }
  for (const StageBlock &b : drop) (void)hipHostFree(b.p);
}

// A block of at least `want` bytes, `want` clamped to [kStageMinBytes, kStageMaxBytes].
class Stage {
 public:
  explicit Stage(size_t want) {
    want = std::min(std::max(want, kStageMinBytes), kStageMaxBytes);
    {
      std::lock_guard<std::mutex> lock(g_stage_mutex);
      for (size_t k = 0; k < g_stage.size(); ++k) {
        if (g_stage[k].bytes < want) continue;
        b_ = g_stage[k];
        g_stage.erase(g_stage.begin() + (std::ptrdiff_t)k);
        return;
      }
    }
    size_t bytes = kStageMinBytes;
    while (bytes < want) bytes *= 2;
    if (hipHostMalloc(&b_.p, bytes, hipHostMallocPortable) != hipSuccess) {
      (void)hipGetLastError();
      fail(SNN_E_OOM, "pinned host allocation of " + std::to_string(bytes) + " bytes failed");
    }
    b_.bytes = bytes;
  }
  ~Stage() {
    StageBlock drop = b_;
    try {
      std::lock_guard<std::mutex> lock(g_stage_mutex);
      if (g_stage.size() < kStageKeep) {
        g_stage.push_back(b_);
        drop.p = nullptr;
      } else {
        // keep the larger blocks
        for (StageBlock &k : g_stage)
          if (k.bytes < drop.bytes) std::swap(k, drop);
      }
    } catch (...) {
    }
    if (drop.p) (void)hipHostFree(drop.p);
  }
  Stage(const Stage &) = delete;
  Stage &operator=(const Stage &) = delete;
  unsigned char *data() const { return static_cast<unsigned char *>(b_.p); }
  size_t bytes() const { return b_.bytes; }

 private:
  StageBlock b_;
};

// ---- pinned slots ---------------------------------------------------------------------
// A few numbers each that a plan's passes leave for the host.  Slots come from 4 KiB blocks, as many
// as the most plans at a time need, and stay mapped when their plan is closed: a pass on a
// caller's stream may still write one.  snn_memory_cache_release returns the blocks when no
// plan has a slot, after the device has drained.
constexpr size_t kSlotBlock = 4096, kSlotBytes = 64;
std::mutex g_slot_mutex;
std::vector<unsigned char *> g_slot_blocks;
std::vector<uint32_t *> g_slots;  // free ones

uint32_t *slot_take() {
  std::lock_guard<std::mutex> lock(g_slot_mutex);
  if (g_slots.empty()) {
    g_slot_blocks.reserve(g_slot_blocks.size() + 1);
    g_slots.reserve((g_slot_blocks.size() + 1) * (kSlotBlock / kSlotBytes));  // giving back cannot fail
    void *p = nullptr;
    check(hipHostMalloc(&p, kSlotBlock, hipHostMallocPortable), "pinned slots");
    g_slot_blocks.push_back(static_cast<unsigned char *>(p));
    for (size_t k = kSlotBlock; k > 0; k -= kSlotBytes)
      g_slots.push_back(reinterpret_cast<uint32_t *>(g_slot_blocks.back() + k - kSlotBytes));
  }
  uint32_t *slot = g_slots.back();
  g_slots.pop_back();
  std::memset(slot, 0, kSlotBytes);
  return slot;
}

void slot_give(uint32_t *slot) {
  std::lock_guard<std::mutex> lock(g_slot_mutex);
  g_slots.push_back(slot);
}

void slot_release() {
  std::lock_guard<std::mutex> lock(g_slot_mutex);
  if (g_slot_blocks.empty() || g_slots.size() != g_slot_blocks.size() * (kSlotBlock / kSlotBytes)) return;
  if (hipDeviceSynchronize() != hipSuccess) return;
  for (unsigned char *p : g_slot_blocks) (void)hipHostFree(p);
  g_slot_blocks.clear();
  g_slots.clear();
}

// ---- streams -------------------------------------------------------------------------
// Networks, batches and plans without a caller's stream have one of their own.  Making and destroying one takes
// about 50 us each, so up to kStreamKeep idle ones are kept; snn_memory_cache_release destroys
// them.
constexpr size_t kStreamKeep = 8;
struct IdleStream {
  int device;
  hipStream_t stream;
};
std::mutex g_stream_mutex;
std::vector<IdleStream> g_streams;

hipStream_t stream_take(int device) {
  {
    std::lock_guard<std::mutex> lock(g_stream_mutex);
    for (size_t k = 0; k < g_streams.size(); ++k) {
      if (g_streams[k].device != device) continue;
      hipStream_t s = g_streams[k].stream;
      g_streams.erase(g_streams.begin() + (std::ptrdiff_t)k);
      return s;
    }
  }
  hipStream_t s = nullptr;
  check(hipStreamCreateWithFlags(&s, hipStreamNonBlocking), "hipStreamCreate");
  return s;
}

// Back after everything on it has run without an error (`clean`).
void stream_give(int device, hipStream_t s, bool clean) {
  if (clean) {
    try {
      std::lock_guard<std::mutex> lock(g_stream_mutex);
      if (g_streams.size() < kStreamKeep) {
        g_streams.push_back({device, s});
        return;
      }
    } catch (...) {
    }
  }
  (void)hipStreamDestroy(s);
}

void stream_release(int device) {
  std::vector<hipStream_t> drop;
  {
    std::lock_guard<std::mutex> lock(g_stream_mutex);
    for (size_t k = g_streams.size(); k-- > 0;) {
      if (device >= 0 && g_streams[k].device != device) continue;
      drop.push_back(g_streams[k].stream);
      g_streams.erase(g_streams.begin() + (std::ptrdiff_t)k);
    }
  }
  for (hipStream_t s : drop) (void)hipStreamDestroy(s);
}

void *dev_alloc(snn_network *net, size_t bytes) {
  if (bytes == 0) bytes = 16;
  bytes = (bytes + 255) & ~(size_t)255;
  void *p = nullptr;
  if (net->has_alloc) {
    p = net->alloc.alloc(bytes, (void *)net->stream, net->alloc.ctx);
    if (!p) fail(SNN_E_OOM, "allocator callback returned NULL for " + std::to_string(bytes) + " bytes");
  } else {
    size_t got = bytes;
    p = pool_alloc(net->device, bytes, &got);
    if (!p) fail(SNN_E_OOM, "hipMalloc of " + std::to_string(bytes) + " bytes failed");
    bytes = got;  // a reused block may be larger than the request: record what is held
  }
  net->allocs.push_back({p, bytes});
  net->device_bytes += bytes;
  return p;
}

template <typename T>
T *dev_array(snn_network *net, size_t count) {
  return static_cast<T *>(dev_alloc(net, count * sizeof(T)));
}

void release(snn_network *net) {
  const bool clean = net->stream && hipStreamSynchronize(net->stream) == hipSuccess;
  if (net->graph) (void)hipGraphExecDestroy(net->graph);
  for (auto &a : net->allocs) {
    if (net->has_alloc) net->alloc.free(a.p, a.bytes, (void *)net->stream, net->alloc.ctx);
    else pool_free(net->device, a.p, a.bytes);
  }
  net->allocs.clear();
  std::vector<hipEvent_t> pend;
  for (auto &r : net->prof_pending) {
    pend.push_back(r.a);
    pend.push_back(r.b);
  }
  std::sort(pend.begin(), pend.end());
  pend.erase(std::unique(pend.begin(), pend.end()), pend.end());
  for (hipEvent_t e : pend) (void)hipEventDestroy(e);
  net->prof_pending.clear();
  for (hipEvent_t e : net->event_pool) (void)hipEventDestroy(e);
  net->event_pool.clear();
  if (net->own_stream && net->stream) stream_give(net->device, net->stream, clean);
}

// ---- definitions of the derived constants -----------------------------------------
int32_t q16(double w_mV, const char *what) {
  const double s = std::nearbyint(w_mV * 65536.0);
  if (!(s > -2147483648.0 && s < 2147483647.0)) fail(SNN_E_INVALID, std::string(what) + " out of Q16 range");
  return (int32_t)s;
}

// Inverse-CDF thresholds of Binomial(n, p): tbl[j] = floor(CDF(j) 2^32) until the
// first index past the mean whose probability is below 2^-40 (or n), which gets 2^32.
// pmf(0) = q^n by n multiplications; pmf(j) = pmf(j-1) (n-j+1) / j (p/q).
uint32_t binomial_thresholds(uint32_t n, double p, uint64_t *tbl, uint32_t cap) {
  const uint64_t kOne = 1ull << 32;
  if (n == 0 || p <= 0.0) {
    tbl[0] = kOne;
    return 1;
  }
  if (p >= 1.0) {
    if (n + 1 > cap) return 0;
    std::fill(tbl, tbl + n, 0ull);
    tbl[n] = kOne;
    return n + 1;
  }
  const double q = 1.0 - p, ratio = p / q, mean = (double)n * p;
  double pmf = 1.0;
  for (uint32_t j = 0; j < n; ++j) pmf *= q;
  if (!(pmf > 0.0)) return 0;
  double cdf = pmf;
  for (uint32_t j = 0;; ++j) {
    if (j + 1 > cap) return 0;
    if (j == n || ((double)j > mean && pmf < 0x1p-40)) {
      tbl[j] = kOne;
      return j + 1;
    }
    const double scaled = cdf * 4294967296.0;
    tbl[j] = scaled >= 4294967296.0 ? kOne : (uint64_t)scaled;
    pmf *= (double)(n - j);  // (n - (j+1) + 1)
    pmf /= (double)(j + 1);
    pmf *= ratio;
    cdf += pmf;
  }
}

void validate_and_derive(snn_network *net) {
  const snn_params &p = net->prm;
  if (!(p.dt_ms > 0.0)) fail(SNN_E_INVALID, "dt_ms must be > 0");
  if (p.delay_steps < 1) fail(SNN_E_INVALID, "delay_steps must be >= 1");
  if (p.synapse_weights > 1) fail(SNN_E_INVALID, "synapse_weights must be 0 (auto) or 1 (per synapse)");
  if (p.plasticity > SNN_PLASTICITY_LAZY) fail(SNN_E_INVALID, "plasticity must be SNN_PLASTICITY_EAGER or _LAZY");
  if (!(p.tau_m_ms > 0.0)) fail(SNN_E_INVALID, "tau_m_ms must be > 0");
  if (!(p.t_ref_ms >= 0.0)) fail(SNN_E_INVALID, "t_ref_ms must be >= 0");
  if (net->pops.empty()) fail(SNN_E_INVALID, "no populations");
  uint64_t n = 0;
  net->pop_off.assign(1, 0u);
  for (const auto &pop : net->pops) {
    if (pop.size == 0) fail(SNN_E_INVALID, "empty population");
    n += pop.size;
    if (n >= (1ull << 31)) fail(SNN_E_INVALID, "too many neurons (>= 2^31)");
    net->pop_off.push_back((uint32_t)n);
  }
  net->n = (uint32_t)n;
  const uint32_t n_pops = (uint32_t)net->pops.size();
  bool plastic = false;
  for (size_t q = 0; q < net->proj.size(); ++q) {
    const snn_projection &pj = net->proj[q];
    const uint32_t span = pj.to_span ? pj.to_span : 1u;
    if (pj.from >= n_pops || pj.to >= n_pops || span > n_pops - pj.to)
      fail(SNN_E_INVALID, "projection " + std::to_string(q) + ": bad population index");
    for (size_t r = 0; r < q; ++r) {
      const snn_projection &o = net->proj[r];
      const uint32_t os = o.to_span ? o.to_span : 1u;
      if (o.from == pj.from && o.to < pj.to + span && pj.to < o.to + os)
        fail(SNN_E_INVALID, "projections " + std::to_string(r) + " and " + std::to_string(q) +
                                " overlap (same source, overlapping targets)");
    }
    (void)q16(pj.w_mV, "weight");
    const uint64_t tsize = (uint64_t)net->pop_off[pj.to + span] - net->pop_off[pj.to];
    const bool self_in = pj.from >= pj.to && pj.from < pj.to + span;
    const uint64_t cand = tsize - (self_in ? 1u : 0u);
    if (pj.kind == SNN_PROJ_ER) {
      if (!(pj.p >= 0.0 && pj.p <= 1.0)) fail(SNN_E_INVALID, "ER probability outside [0, 1]");
    } else if (pj.kind == SNN_PROJ_FIXED_OUT) {
      if (pj.k > cand) fail(SNN_E_INVALID, "out-degree exceeds the number of candidate targets");
      const uint64_t spare = cand - pj.k;
      if (((uint64_t)pj.k + 1) * (2 * spare + 1) > (1ull << 35))
        fail(SNN_E_INVALID, "out-degree x target range too large for exact 64-bit spacing");
    } else {
      fail(SNN_E_INVALID, "unknown projection kind");
    }
    if (pj.plastic) {
      plastic = true;
      for (size_t r = 0; r < net->proj.size(); ++r)
        if (r != q && net->proj[r].plastic && net->proj[r].from == pj.from)
          fail(SNN_E_INVALID, "at most one plastic projection per source population");
    }
  }
  net->plastic = plastic;
  net->lazy = plastic && p.plasticity == SNN_PLASTICITY_LAZY;
  if (net->lazy && p.delay_steps > snn::kLazyHistory)
    fail(SNN_E_INVALID, "lazy plasticity needs delay_steps <= " + std::to_string(snn::kLazyHistory));
  net->delay = p.delay_steps;
  net->alpha = (float)std::exp(-p.dt_ms / p.tau_m_ms);
  net->v_inf = (float)(p.v_rest_mV + p.v_bg_mV);
  net->v_th = (float)p.v_th_mV;
  net->v_reset = (float)p.v_reset_mV;
  const double rs = std::nearbyint(p.t_ref_ms / p.dt_ms);
  if (rs > 1e9) fail(SNN_E_INVALID, "refractory period too long");
  net->ref_steps = (int32_t)rs;
  net->w_ext_q16 = q16(p.w_ext_mV, "w_ext");
  if (plastic) {
    if (!(p.tau_plus_ms > 0.0 && p.tau_minus_ms > 0.0)) fail(SNN_E_INVALID, "STDP time constants must be > 0");
    if (!(p.w_max_mV >= 0.0)) fail(SNN_E_INVALID, "w_max must be >= 0");
    net->beta_plus = (float)std::exp(-p.dt_ms / p.tau_plus_ms);
    net->beta_minus = (float)std::exp(-p.dt_ms / p.tau_minus_ms);
    net->a_plus = (float)p.a_plus;
    net->a_minus = (float)p.a_minus;
    net->w_max = (float)p.w_max_mV;
  }
  const double p_ext = (p.rate_ext_hz * p.dt_ms) / 1000.0;
  if (p.n_ext > 0 && !(p_ext >= 0.0 && p_ext <= 1.0)) fail(SNN_E_INVALID, "drive rate x dt outside [0, 1]");
  net->table_len = binomial_thresholds(p.n_ext, p_ext, net->table, snn::kTableCap);
  if (net->table_len == 0) fail(SNN_E_INVALID, "drive distribution needs more than 256 table entries");
  net->key0 = (uint32_t)p.seed;
  net->key1 = (uint32_t)(p.seed >> 32);
}

// ---- schedule: window, FIFO sizes, delivery variant --------------------------------
void choose_schedule(snn_network *net) {
  const snn_params &p = net->prm;
  if (net->plastic) {
    // Synapses change every step and delivery must see Syn_{t+1}: deliver S_{t-d+1}
    // at step t into a single accumulator (the paper's schedule).
    net->window = 1;
    net->n_inbuf = 1;
    // lazy plasticity delivers inside its own kernel (the atomic kernel serves only
    // delivery timing); eager plasticity takes either delivery, one step per launch
    if (net->lazy && p.delivery == SNN_DELIVERY_TILED)
      fail(SNN_E_INVALID, "lazy plasticity delivers inside its own kernel; tiled delivery needs eager plasticity");
    net->delivery = net->lazy ? SNN_DELIVERY_ATOMIC : p.delivery;
  } else {
    // Static weights: a spike of step e may be delivered any time between the updates
    // of e and e + d; one accumulator per pending arrival step lets a window of up to
    // d updates run in one launch, followed by one delivery launch for its queues.
    net->n_inbuf = net->delay;
    net->window = p.window ? std::min(p.window, net->delay) : net->delay;
    net->window = std::min(net->window, 64u);  // one ballot per lane of the update wave
    net->delivery = p.delivery;
  }
  net->raster_cap = p.raster_steps ? p.raster_steps : 1024u;
  // eager STDP reads the spike bits of step t - d from the raster ring
  if (net->plastic) net->raster_cap = std::max(net->raster_cap, net->delay + 1);
  net->window = std::min(net->window, net->raster_cap);  // kernels step rings by one wrap
  net->slots = std::max(net->delay + 2, 2 * net->window);
  net->words = (net->n + 63) / 64;
}

void choose_delivery(snn_network *net) {
  if (net->delivery == SNN_DELIVERY_AUTO) {
    const double deg = net->n ? (double)net->nnz / net->n : 0.0;
    net->delivery = (net->n >= 16384 && deg >= 64.0) ? SNN_DELIVERY_TILED : SNN_DELIVERY_ATOMIC;
  }
  if (net->delivery == SNN_DELIVERY_TILED) {
    const uint32_t b = net->prm.block;
    if (b != 0 && b != 256 && b != 512 && b != 1024) fail(SNN_E_INVALID, "block must be 256, 512 or 1024");
    net->block = b ? b : 1024;
    // A workgroup accumulates a range of up to kTileGroupMax base tiles in LDS.  The
    // largest base tile is set by the workgroup LDS limit (160 KB on gfx950, less the
    // kernel's static arrays); the default base tile is kDefaultTile targets, so that a
    // range holds up to 18,432 targets (the fastest range size of the launch-shape sweep
    // on the 1e9-synapse network, with 1,024-thread workgroups and one per CU).  Small
    // base tiles let the schedule size ranges in steps of 1/32 of that.
    size_t lds_dyn = 0;
    check(snn::prepare_deliver_tiled(net->block, &lds_dyn), "tiled delivery LDS limit");
    // a range's accumulators fit the LDS, and the delivery reads 16-bit targets, which
    // identify a target only inside a range of fewer than 65,536 targets
    const uint64_t range_cap = std::min<uint64_t>(lds_dyn / 4, 65535);
    constexpr uint32_t kDefaultTile = 576;
    const uint32_t tile_cap = (uint32_t)(range_cap / snn::kTileGroupMax);
    const uint32_t min_tiles = net->n <= range_cap ? 1u : (net->n + tile_cap - 1) / tile_cap;
    uint32_t tiles = net->prm.tiles ? net->prm.tiles : (net->n + kDefaultTile - 1) / kDefaultTile;
    tiles = std::max(std::min(tiles, std::max(1u, net->n / 16u)), min_tiles);
    // a multiple of 4 targets, so that ranges start on 16-byte boundaries of a row of
    // accumulators (the range flush then stores 16 bytes at a time)
    net->tile_size = ((net->n + tiles - 1) / tiles + 3) & ~3u;
    net->tiles = (net->n + net->tile_size - 1) / net->tile_size;
    if ((uint64_t)std::min(net->tiles, snn::kTileGroupMax) * net->tile_size > range_cap)
      fail(SNN_E_INVALID, "tile range too large for LDS or for 16-bit targets");
    // one 1,024-thread workgroup per CU (the kernel's registers allow one resident)
    net->grid = net->prm.grid ? net->prm.grid : net->cu_count * (net->block == 1024 ? 1u : 2u);
  } else if (net->delivery == SNN_DELIVERY_ATOMIC) {
    net->tiles = 1;
    net->tile_size = net->n;
  } else {
    fail(SNN_E_INVALID, "unknown delivery variant");
  }
}

// ---- construction ----------------------------------------------------------------
hipEvent_t new_event() {
  hipEvent_t e;
  // timing markers only: no system-scope fence when the event is recorded, so that a
  // marker between two launches costs as little as possible
  check(hipEventCreateWithFlags(&e, hipEventDisableSystemFence), "hipEventCreate");
  return e;
}

// Indexes of the tiled delivery: the tile boundaries of every row (uint16 when no row can
// reach 65,536 synapses, else uint32) and the 16-bit copy of the targets it streams.
snn::RowIndex alloc_tile_offsets(snn_network *net) {
  const uint64_t count = ((net->nnz + 7) & ~7ull) + 8;  // whole 16-byte groups, one spare
  if (!net->col16) net->col16 = dev_array<uint16_t>(net, count);
  net->tile_off16 = net->row_len_bound < 65536;
  const size_t entries = (size_t)net->n * (net->tiles + 1);
  if (net->tile_off16) net->tile_off = dev_array<uint16_t>(net, entries);
  else net->tile_off = dev_array<uint32_t>(net, entries);
  return {net->col16, net->tile_off, net->nnz, count, net->tiles, net->tile_size, net->tile_off16, 0u};
}

void fill_tile_offsets(snn_network *net, const snn::RowIndex &x) {
  check(snn::launch_tile_index(net->row_ptr, net->col, net->n, x.nnz, x.count, x.tiles, x.tile_size, x.col16,
                               x.tile_off, x.off16, net->stream),
        "tile index");
}

bool choose_solo(const snn_network *net);
bool choose_windows(snn_network *net);

void build(snn_network *net) {
  validate_and_derive(net);
  choose_schedule(net);
  hipStream_t s = net->stream;
  const uint32_t n = net->n, n_pops = (uint32_t)net->pops.size();

  // projections grouped by source population, sorted by first target population
  std::vector<snn::GenProj> gp;
  std::vector<uint32_t> pop_proj(n_pops + 1, 0);
  for (uint32_t a = 0; a < n_pops; ++a) {
    std::vector<const snn_projection *> mine;
    for (const auto &pj : net->proj)
      if (pj.from == a) mine.push_back(&pj);
    std::sort(mine.begin(), mine.end(), [](auto *x, auto *y) { return x->to < y->to; });
    pop_proj[a] = (uint32_t)gp.size();
    for (const snn_projection *pj : mine) {
      const uint32_t span = pj->to_span ? pj->to_span : 1u;
      snn::GenProj g{};
      g.kind = pj->kind;
      g.k = pj->k;
      g.first_pop = pj->to;
      g.off = net->pop_off[pj->to];
      g.size = net->pop_off[pj->to + span] - g.off;
      g.self_in = (a >= pj->to && a < pj->to + span) ? 1u : 0u;
      g.plastic = pj->plastic ? 1u : 0u;
      g.w_q16 = q16(pj->w_mV, "weight");
      g.w_f32 = (float)pj->w_mV;
      g.thr = pj->p >= 1.0 ? (1ull << 32) : (uint64_t)(pj->p * 4294967296.0);
      g.spare = pj->kind == SNN_PROJ_FIXED_OUT ? (uint64_t)(g.size - g.self_in - pj->k) : 0;
      gp.push_back(g);
    }
  }
  pop_proj[n_pops] = (uint32_t)gp.size();
  // longest possible row: a source's fixed out-degrees plus the sizes of the target
  // ranges of its ER projections
  net->row_len_bound = 0;
  for (uint32_t a = 0; a < n_pops; ++a) {
    uint64_t b = 0;
    for (uint32_t q = pop_proj[a]; q < pop_proj[a + 1]; ++q)
      b += gp[q].kind == SNN_PROJ_FIXED_OUT ? gp[q].k : gp[q].size;
    net->row_len_bound = std::max(net->row_len_bound, b);
  }

  snn::GenProj *d_proj = dev_array<snn::GenProj>(net, std::max<size_t>(gp.size(), 1));
  uint32_t *d_pop_off = dev_array<uint32_t>(net, n_pops + 1);
  uint32_t *d_pop_proj = dev_array<uint32_t>(net, n_pops + 1);
  if (!gp.empty())
    check(hipMemcpyAsync(d_proj, gp.data(), gp.size() * sizeof(snn::GenProj), hipMemcpyHostToDevice, s), "copy projections");
  check(hipMemcpyAsync(d_pop_off, net->pop_off.data(), (n_pops + 1) * 4, hipMemcpyHostToDevice, s), "copy offsets");
  check(hipMemcpyAsync(d_pop_proj, pop_proj.data(), (n_pops + 1) * 4, hipMemcpyHostToDevice, s), "copy ranges");
  snn::GenArgs g{d_proj, d_pop_off, d_pop_proj, n_pops, n, net->key0, net->key1};

  // row lengths -> row pointers -> rows
  uint32_t *len = dev_array<uint32_t>(net, n);
  if (net->plastic) {
    net->plast_rel = dev_array<uint32_t>(net, n);
    net->plast_len = dev_array<uint32_t>(net, n);
  }
  // setup timing: HIP events on the build stream around the generation phases
  hipEvent_t ev[6];
  for (hipEvent_t &e : ev) e = new_event();
  struct EventGuard {
    hipEvent_t *e;
    ~EventGuard() {
      for (int k = 0; k < 6; ++k) (void)hipEventDestroy(e[k]);
    }
  } ev_guard{ev};
  check(hipEventRecord(ev[0], s), "hipEventRecord");
  check(snn::launch_row_lengths(g, len, net->plast_rel, net->plast_len, s), "row lengths");
  net->row_ptr = dev_array<uint64_t>(net, (size_t)n + 1);
  uint64_t *scan_tmp = dev_array<uint64_t>(net, snn::scan_scratch_elems(n));
  check(snn::launch_scan_u32_to_u64(len, net->row_ptr, n, scan_tmp, s), "row scan");
  check(hipEventRecord(ev[1], s), "hipEventRecord");
  uint32_t max_fixed_k = 0;
  bool all_fixed = true;
  for (const snn::GenProj &q : gp) {
    if (q.kind == SNN_PROJ_FIXED_OUT) max_fixed_k = std::max(max_fixed_k, q.k);
    else all_fixed = false;
  }
  if (all_fixed) {  // the number of synapses is known without the scan
    net->nnz = 0;
    for (uint32_t a = 0; a < n_pops; ++a)
      for (uint32_t q = pop_proj[a]; q < pop_proj[a + 1]; ++q)
        net->nnz += (uint64_t)(net->pop_off[a + 1] - net->pop_off[a]) * gp[q].k;
  } else {
    check(hipMemcpyAsync(&net->nnz, net->row_ptr + n, sizeof(uint64_t), hipMemcpyDeviceToHost, s), "read nnz");
    check(hipStreamSynchronize(s), "sync after row scan");
  }
  if (net->plastic && net->nnz >= (1ull << 32)) fail(SNN_E_INVALID, "plastic networks are limited to 2^32 synapses");
  net->nnz_alloc = ((net->nnz + 3) & ~3ull) + 4;  // 16-byte groups of the atomic delivery
  net->col = dev_array<int32_t>(net, net->nnz_alloc);
  // the fill writes every synapse: only the padding past the last one is cleared here
  const size_t pad_bytes = (net->nnz_alloc - net->nnz) * 4;
  check(hipMemsetAsync(net->col + net->nnz, 0, pad_bytes, s), "clear col padding");
  // Table I layout: when every projection from a source population carries the same
  // weight, a synapse stores only its target and the weight is the source's
  bool src_uniform = !net->plastic && net->prm.synapse_weights == 0;
  std::vector<int32_t> pop_w(n_pops, 0);
  for (uint32_t a = 0; a < n_pops && src_uniform; ++a) {
    bool seen = false;
    for (uint32_t q = pop_proj[a]; q < pop_proj[a + 1]; ++q) {
      if (seen && gp[q].w_q16 != pop_w[a]) src_uniform = false;
      pop_w[a] = gp[q].w_q16;
      seen = true;
    }
  }
  if (net->plastic) {
    net->w_f32 = dev_array<float>(net, net->nnz_alloc);
    check(hipMemsetAsync(net->w_f32 + net->nnz, 0, pad_bytes, s), "clear w padding");
  } else if (src_uniform) {
    net->w_src_host.assign(n, 0);
    for (uint32_t a = 0; a < n_pops; ++a)
      std::fill(net->w_src_host.begin() + net->pop_off[a], net->w_src_host.begin() + net->pop_off[a + 1], pop_w[a]);
    net->w_src = dev_array<int32_t>(net, n);
    check(hipMemcpyAsync(net->w_src, net->w_src_host.data(), (size_t)n * 4, hipMemcpyHostToDevice, s),
          "copy source weights");
  } else {
    net->w_q16 = dev_array<int32_t>(net, net->nnz_alloc);
    check(hipMemsetAsync(net->w_q16 + net->nnz, 0, pad_bytes, s), "clear w padding");
  }
  choose_delivery(net);
  net->delivery_chosen = net->prm.delivery != SNN_DELIVERY_AUTO || net->prm.tiles || net->prm.block || net->prm.grid;
  net->solo = choose_solo(net);
  snn::RowIndex index{};
  if (net->delivery == SNN_DELIVERY_TILED) index = alloc_tile_offsets(net);
  // rows of one fixed out-degree projection get their indexes while they are filled
  bool one_each = all_fixed;
  for (uint32_t a = 0; a < n_pops; ++a) one_each = one_each && pop_proj[a + 1] - pop_proj[a] <= 1;
  check(hipEventRecord(ev[2], s), "hipEventRecord");
  check(snn::launch_fill_rows(g, max_fixed_k, all_fixed, net->row_ptr, net->col, net->w_q16, net->w_f32,
                              one_each ? index : snn::RowIndex{}, s),
        "fill rows");
  check(hipEventRecord(ev[3], s), "hipEventRecord");
  check(hipEventRecord(ev[4], s), "hipEventRecord");

  if (net->plastic) {
    // plastic in-edges grouped by target: counting sort by target
    uint32_t *cnt = dev_array<uint32_t>(net, n);
    check(hipMemsetAsync(cnt, 0, (size_t)n * 4, s), "clear in-degree");
    check(snn::launch_count_in_edges(net->row_ptr, net->col, net->plast_rel, net->plast_len, n, cnt, s), "count in-edges");
    net->in_ptr = dev_array<uint64_t>(net, (size_t)n + 1);
    check(snn::launch_scan_u32_to_u64(cnt, net->in_ptr, n, scan_tmp, s), "in-edge scan");
    uint64_t n_in = 0;
    check(hipMemcpyAsync(&n_in, net->in_ptr + n, 8, hipMemcpyDeviceToHost, s), "read plastic count");
    check(hipStreamSynchronize(s), "sync");
    net->in_src = dev_array<int32_t>(net, std::max<uint64_t>(n_in, 1));
    net->in_edge = dev_array<uint32_t>(net, std::max<uint64_t>(n_in, 1));
    uint64_t *cursor = dev_array<uint64_t>(net, n);
    check(hipMemcpyAsync(cursor, net->in_ptr, (size_t)n * 8, hipMemcpyDeviceToDevice, s), "cursor");
    check(snn::launch_fill_in_edges(net->row_ptr, net->col, net->plast_rel, net->plast_len, n, cursor,
                                    net->in_src, net->in_edge, s), "fill in-edges");
  }

  if (index.col16 && !one_each) fill_tile_offsets(net, index);
  check(hipEventRecord(ev[5], s), "hipEventRecord");

  // neuron state, FIFO, raster, control block
  net->v = dev_array<float>(net, n);
  net->ref = dev_array<int32_t>(net, n);
  net->input = dev_array<int32_t>(net, (size_t)net->n_inbuf * n);
  net->x_pre = dev_array<float>(net, n);
  net->x_post = dev_array<float>(net, n);
  // spike queues: kQueueGroups sub-queues per slot, sub-queue g collecting the spikes
  // of update workgroups b with b % kQueueGroups == g
  const uint32_t upd_blocks = (n + snn::kUpdateBlock - 1) / snn::kUpdateBlock;
  net->group_cap = ((upd_blocks + snn::kQueueGroups - 1) / snn::kQueueGroups) * snn::kUpdateBlock;
  net->queue_stride = snn::kQueueGroups * net->group_cap;
  net->queue = dev_array<int32_t>(net, (size_t)net->slots * net->queue_stride);
  net->qlen = dev_array<uint32_t>(net, (size_t)net->slots * snn::kQueueGroups * snn::kQlenStride);
  // the raster ring, and behind it the offsets scratch of the spike download
  const size_t ring_words = (size_t)net->raster_cap * net->words;
  net->raster_scratch = snn::raster_scratch(ring_words);
  net->raster = dev_array<uint64_t>(net, ring_words + net->raster_scratch);
  net->raster_offset = net->raster + ring_words;
  net->d_table32 = dev_array<uint32_t>(net, snn::kTableCap);
  net->d_guide = dev_array<uint16_t>(net, snn::kGuideBuckets);
  net->ctl = dev_array<snn::Ctl>(net, 1);
  check(hipMemsetAsync(net->input, 0, (size_t)net->n_inbuf * n * 4, s), "clear input");
  check(hipMemsetAsync(net->x_pre, 0, (size_t)n * 4, s), "clear traces");
  check(hipMemsetAsync(net->x_post, 0, (size_t)n * 4, s), "clear traces");
  check(hipMemsetAsync(net->qlen, 0, (size_t)net->slots * snn::kQueueGroups * snn::kQlenStride * 4, s),
        "clear queues");
  check(hipMemsetAsync(net->raster, 0, (size_t)net->raster_cap * net->words * 8, s), "clear raster");
  check(hipMemsetAsync(net->ctl, 0, sizeof(snn::Ctl), s), "clear control");
  if (net->lazy) {
    // Rows start with nothing pending and ages spread over the history, so that as many
    // rows expire at every step: row i's first pending step is -(i mod 64), before which
    // no event exists (empty histories, zero traces).
    net->hist = dev_array<uint64_t>(net, n);
    net->age = dev_array<uint32_t>(net, n);
    net->x_age = dev_array<float>(net, n);
    net->exq = dev_array<int32_t>(net, 2 * (size_t)net->queue_stride);
    net->exq_len = dev_array<uint32_t>(net, 2 * (size_t)snn::kQueueGroups * snn::kQlenStride);
    check(hipMemsetAsync(net->hist, 0, (size_t)n * 8, s), "clear spike history");
    check(hipMemsetAsync(net->x_age, 0, (size_t)n * 4, s), "clear traces at age");
    check(hipMemsetAsync(net->exq_len, 0, 2 * (size_t)snn::kQueueGroups * snn::kQlenStride * 4, s),
          "clear expiring rows");
    std::vector<uint32_t> age0(n);
    for (uint32_t i = 0; i < n; ++i) age0[i] = 0u - (i % snn::kLazyHistory);
    check(hipMemcpyAsync(net->age, age0.data(), (size_t)n * 4, hipMemcpyHostToDevice, s), "row ages");
    check(hipStreamSynchronize(s), "sync");
  }
  // the drive table as the kernels search it: thresholds below 2^32 as 32-bit words, and
  // a guide table giving #{j : tbl[j] <= r} at both ends of each bucket of r's top bits
  {
    std::vector<uint32_t> t32(snn::kTableCap, 0u);
    uint32_t below = 0;
    while (below < net->table_len && net->table[below] < (1ull << 32)) {
      t32[below] = (uint32_t)net->table[below];
      ++below;
    }
    std::vector<uint16_t> guide(snn::kGuideBuckets);
    const uint32_t shift = 32 - snn::kGuideBits;
    for (uint32_t b = 0; b < snn::kGuideBuckets; ++b) {
      const uint64_t r_lo = (uint64_t)b << shift, r_hi = r_lo + ((1ull << shift) - 1);
      uint32_t lo = 0, hi = 0;
      for (uint32_t j = 0; j < below; ++j) {
        lo += t32[j] <= r_lo ? 1u : 0u;
        hi += t32[j] <= r_hi ? 1u : 0u;
      }
      guide[b] = (uint16_t)(lo | (hi << 8));
    }
    check(hipMemcpyAsync(net->d_table32, t32.data(), t32.size() * 4, hipMemcpyHostToDevice, s), "copy table");
    check(hipMemcpyAsync(net->d_guide, guide.data(), guide.size() * 2, hipMemcpyHostToDevice, s), "copy guide");
    check(hipStreamSynchronize(s), "sync tables");
  }
  const float lo = (float)net->prm.v0_lo_mV;
  const float span = (float)(net->prm.v0_hi_mV - net->prm.v0_lo_mV);
  check(snn::launch_init_neurons(net->v, net->ref, n, net->key0, net->key1, lo, span, s), "init neurons");
  // after everything the network cannot do without: the windows' buffers take what is left
  net->windows = choose_windows(net);
  check(hipStreamSynchronize(s), "sync after build");
  check(hipEventElapsedTime(&net->gen_rows_ms, ev[0], ev[1]), "hipEventElapsedTime");
  check(hipEventElapsedTime(&net->gen_fill_ms, ev[2], ev[3]), "hipEventElapsedTime");
  check(hipEventElapsedTime(&net->index_ms, ev[4], ev[5]), "hipEventElapsedTime");
}

// ---- the step pipeline --------------------------------------------------------------
snn::QueueRef queue_ref(snn_network *net) {
  return snn::QueueRef{net->queue, net->qlen, net->queue_stride, net->group_cap};
}

snn::LazyRef lazy_ref(snn_network *net) {
  snn::LazyRef r{};
  r.hist = net->hist;
  r.age = net->age;
  r.x_age = net->x_age;
  r.plast_len = net->plast_len;
  r.exq = snn::QueueRef{net->exq, net->exq_len, net->queue_stride, net->group_cap};
  r.delay = net->delay;
  return r;
}

snn::UpdateArgs update_args(snn_network *net) {
  snn::UpdateArgs a{};
  a.v = net->v;
  a.ref = net->ref;
  a.input = net->input;
  a.x_pre = net->x_pre;
  a.x_post = net->x_post;
  a.q = queue_ref(net);
  a.raster = net->raster;
  a.table32 = net->d_table32;
  a.guide = net->d_guide;
  a.ctl = net->ctl;
  a.n = net->n;
  a.slots = net->slots;
  a.n_inbuf = net->n_inbuf;
  a.raster_cap = net->raster_cap;
  a.words = net->words;
  a.table_len = net->table_len;
  a.key0 = net->key0;
  a.key1 = net->key1;
  a.alpha = net->alpha;
  a.v_inf = net->v_inf;
  a.v_th = net->v_th;
  a.v_reset = net->v_reset;
  a.beta_plus = net->beta_plus;
  a.beta_minus = net->beta_minus;
  a.ref_steps = net->ref_steps;
  a.w_ext_q16 = net->w_ext_q16;
  // the tiled delivery overwrites every accumulator it owns; the atomic one adds
  a.zero_input = net->delivery == SNN_DELIVERY_ATOMIC ? 1u : 0u;
  a.plastic = net->plastic ? 1u : 0u;
  if (net->lazy) a.lazy = lazy_ref(net);
  return a;
}

snn::DeliverArgs deliver_args(snn_network *net) {
  snn::DeliverArgs a{};
  a.row_ptr = net->row_ptr;
  a.col = net->col;
  a.w_q16 = net->w_q16;
  a.w_f32 = net->w_f32;
  a.w_src = net->w_src;
  a.q = queue_ref(net);
  a.input = net->input;
  a.col16 = net->col16;
  a.tile_off = net->tile_off;
  a.ctl = net->ctl;
  a.n = net->n;
  a.slots = net->slots;
  a.n_inbuf = net->n_inbuf;
  a.delay = net->delay;
  a.window_max = net->window;
  a.tiles = net->tiles;
  a.tile_size = net->tile_size;
  a.row_groups = (uint32_t)(net->nnz / std::max(1u, net->n) / 8);
  a.off16 = net->tile_off16 ? 1u : 0u;
  a.advance = 1;
  return a;
}

snn::StdpArgs stdp_args(snn_network *net) {
  snn::StdpArgs a{};
  a.row_ptr = net->row_ptr;
  a.col = net->col;
  a.w_f32 = net->w_f32;
  a.plast_rel = net->plast_rel;
  a.plast_len = net->plast_len;
  a.in_ptr = net->in_ptr;
  a.in_src = net->in_src;
  a.in_edge = net->in_edge;
  a.x_pre = net->x_pre;
  a.x_post = net->x_post;
  a.q = queue_ref(net);
  a.ctl = net->ctl;
  a.raster = net->raster;
  a.raster_cap = net->raster_cap;
  a.words = net->words;
  a.n = net->n;
  a.slots = net->slots;
  a.delay = net->delay;
  a.a_plus = net->a_plus;
  a.a_minus = net->a_minus;
  a.w_max = net->w_max;
  return a;
}

snn::LazyArgs lazy_args(snn_network *net) {
  snn::LazyArgs a{};
  a.row_ptr = net->row_ptr;
  a.col = net->col;
  a.w_f32 = net->w_f32;
  a.plast_rel = net->plast_rel;
  a.x_pre = net->x_pre;
  a.x_post = net->x_post;
  a.q = queue_ref(net);
  a.input = net->input;
  a.lazy = lazy_ref(net);
  a.ctl = net->ctl;
  a.n = net->n;
  a.slots = net->slots;
  a.delay = net->delay;
  a.a_plus = net->a_plus;
  a.w_max = net->w_max;
  a.beta_plus = net->beta_plus;
  return a;
}

uint32_t atomic_grid(const snn_network *net) { return net->cu_count * 8; }
uint32_t lazy_grid(const snn_network *net) { return net->cu_count * 4; }

// Lazy plasticity: brings every plastic row current at the step boundary (weights and
// the touch count then equal the eager form's), without changing what the simulation
// computes next.  Ordered on the network's stream.
void lazy_flush(snn_network *net) {
  if (!net->lazy) return;
  check(snn::launch_lazy_flush(lazy_args(net), net->t_host, lazy_grid(net), net->stream), "lazy flush");
}

hipError_t launch_delivery(snn_network *net, const snn::DeliverArgs &d, uint32_t steps,
                           const snn::LaunchEvents &ev = {}) {
  if (net->delivery == SNN_DELIVERY_TILED)
    return snn::launch_deliver_tiled(d, steps, net->block, net->grid, net->stream, ev);
  return snn::launch_deliver_atomic(d, steps, atomic_grid(net), net->stream, ev);
}

hipEvent_t pooled_event(snn_network *net) {
  if (net->event_pool.empty()) return new_event();
  hipEvent_t e = net->event_pool.back();
  net->event_pool.pop_back();
  return e;
}

// With profiling on, every launch gets its own pair of events, stamped by the dispatch
// itself with its begin and end (hipExtLaunchKernel): no marker packet is placed between
// launches, so the durations are the kernels' own and the stream runs as without them.
template <typename F>
void timed(snn_network *net, int kind, F &&launch) {
  if (!net->profiling) {
    check(launch(snn::LaunchEvents{}), "kernel launch");
    return;
  }
  snn::LaunchEvents ev;
  ev.start = pooled_event(net);
  ev.stop = pooled_event(net);
  check(launch(ev), "kernel launch");
  net->prof_pending.push_back(snn_network::ProfRecord{kind, ev.start, ev.stop});
}

void resolve_profile(snn_network *net) {
  auto &v = net->prof_pending;
  if (v.empty()) return;
  check(hipStreamSynchronize(net->stream), "sync");
  std::vector<hipEvent_t> done;
  for (auto &r : v) {
    float ms = 0.f;
    check(hipEventElapsedTime(&ms, r.a, r.b), "hipEventElapsedTime");
    if (r.kind == 0) {
      net->prof.update_ms += ms;
      net->prof.update_launches++;
    } else if (r.kind == 1) {
      net->prof.deliver_ms += ms;
      net->prof.deliver_launches++;
    } else {
      net->prof.stdp_ms += ms;
      net->prof.stdp_launches++;
    }
    done.push_back(r.a);
    done.push_back(r.b);
  }
  std::sort(done.begin(), done.end());
  done.erase(std::unique(done.begin(), done.end()), done.end());
  net->event_pool.insert(net->event_pool.end(), done.begin(), done.end());
  v.clear();
}

// One window of `steps` consecutive steps: update -> [STDP] -> delivery.
void issue_window(snn_network *net, uint32_t steps) {
  const snn::UpdateArgs u = update_args(net);
  timed(net, 0, [&](const snn::LaunchEvents &ev) { return snn::launch_update(u, steps, net->stream, ev); });
  if (net->lazy) {
    // depression over the arriving rows, then one launch for the transmitting rows
    // (pending potentiation, delivery) and the expiring rows
    const snn::StdpArgs sa = stdp_args(net);
    timed(net, 2, [&](const snn::LaunchEvents &ev) { return snn::launch_stdp_ltd(sa, net->cu_count * 4, net->stream, ev); });
    const snn::LazyArgs la = lazy_args(net);
    timed(net, 1, [&](const snn::LaunchEvents &ev) { return snn::launch_lazy(la, lazy_grid(net), net->stream, ev); });
    net->t_host += steps;
    return;
  }
  snn::DeliverArgs d = deliver_args(net);
  if (net->plastic) {
    // depression and potentiation in one pass; the delivery then adds the arrivals to
    // x_pre and S_t to x_post
    const snn::StdpArgs sa = stdp_args(net);
    timed(net, 2, [&](const snn::LaunchEvents &ev) { return snn::launch_stdp_fused(sa, net->cu_count * 4, net->stream, ev); });
    d.x_pre = net->x_pre;
    d.x_post = net->x_post;
  }
  timed(net, 1, [&](const snn::LaunchEvents &ev) { return launch_delivery(net, d, steps, ev); });
  net->t_host += steps;
}

// A high rate (population averages in use lie below it), and the spikes per step at a rate.
constexpr double kLowHz = 15.0, kHighHz = 100.0;
double spikes_at(const snn_network *net, double hz) { return net->n * hz * net->prm.dt_ms * 1e-3; }

// ---- the persistent one-workgroup form -----------------------------------------------
// Drive thresholds a 32-bit word can reach.
uint32_t drive_thresholds(const snn_network *net) {
  uint32_t below = 0;
  while (below < net->table_len && net->table[below] < (1ull << 32)) ++below;
  return below;
}

uint32_t lanes_shift_for(double degree, uint32_t degree_div) {
  const double want = degree / (double)std::max(1u, degree_div);
  uint32_t sh = 0;
  while (sh < 6 && (double)(1u << sh) < want) ++sh;
  return sh;
}

// A static network as the persistent kernels see it.
snn::BatchNet batch_net(snn_network *m) {
  snn::BatchNet d{};
  d.row_ptr = m->row_ptr;
  d.col = m->col;
  d.w_q16 = m->w_q16;
  d.w_src = m->w_src;
  d.v = m->v;
  d.ref = m->ref;
  d.input = m->input;
  d.queue = m->queue;
  d.qlen = m->qlen;
  d.raster = m->raster;
  d.table32 = m->d_table32;
  d.ctl = m->ctl;
  d.n = m->n;
  d.words = m->words;
  d.delay = m->delay;
  d.raster_cap = m->raster_cap;
  d.slots = m->slots;
  d.queue_stride = m->queue_stride;
  d.group_cap = m->group_cap;
  d.window = m->window;
  d.below = drive_thresholds(m);
  d.lanes_shift = lanes_shift_for(m->n ? (double)m->nnz / m->n : 0.0, 4);
  d.key0 = m->key0;
  d.key1 = m->key1;
  d.alpha = m->alpha;
  d.v_inf = m->v_inf;
  d.v_th = m->v_th;
  d.v_reset = m->v_reset;
  d.ref_steps = m->ref_steps;
  d.w_ext_q16 = m->w_ext_q16;
  return d;
}

// LDS of a persistent launch whose largest network needs `need` bytes and has n neurons.
snn::LdsPlan lds_plan(size_t need, uint32_t n, size_t limit) {
  snn::LdsPlan r{};
  r.q_cap = (uint32_t)std::min<size_t>(snn::kBatchQueueMax, (limit - need) / 12);
  r.words = (uint32_t)std::min(limit / 4, need / 4 + 3 * (size_t)r.q_cap + n + 1);
  return r;
}

size_t solo_need(const snn_network *net) { return (size_t)net->delay * net->n * 4; }

// Whether snn_run may step the network by the persistent kernel: a small static network without
// drive, with nothing about its delivery chosen by the caller.  A step of the pipeline costs
// two launches per window of `delay` steps, whatever the size: 6.6-8.9 us with the atomic
// delivery (1,000-40,000 neurons) and 9.6-11.2 us with the tiled one.  A persistent step
// costs about 0.9 us, 0.105 us per 1,000 neurons and 1 us per 8,200 synaptic events: 0.9 us
// at 1,000 neurons, 1.4 at 4,000, 1.9 at 8,000, 3.1 at 16,000, 5.0 at 32,000, against 6.6,
// 7.9, 8.3, 8.6 and 10.9 us (delay 1).  The rule takes 15 Hz for the unknown rate; whether the
// network takes the kernel at the rate it turns out to have is decided below (solo_now).
bool choose_solo(const snn_network *net) {
  if (net->plastic || net->owner || net->delivery_chosen || net->prm.window) return false;
  if (net->n > snn::kSoloMaxNeurons || net->n_inbuf != net->delay || drive_thresholds(net)) return false;
  if (solo_need(net) + snn::kBatchStaticLds > net->lds_limit) return false;
  const double events = (double)net->nnz * kLowHz * net->prm.dt_ms * 1e-3;
  const double step_us = 0.9 + 0.105e-3 * net->n + events / 8200.0;
  return step_us * net->delay <= (net->delivery == SNN_DELIVERY_TILED ? 9.6 : 6.6);
}

// The rule above guesses the rate.  What follows corrects it by the spikes of the network's latest
// steps, which calls that wait for the device anyway find out (note_spikes, measure_spikes).
//
// us per step of the persistent kernel and of the launches (one update and one delivery per
// window) at `spikes` spikes per step.  A spike costs one workgroup 0.02 us and 0.13 ns per synapse; measured, with
// the estimate behind it: 8,000 neurons (800 synapses each) at 56 spikes 7.9 (8.7), at 88 11.0
// (12.7); 16,000 (320) at 100 9.0 (8.7), at 191 15.3 (14.3); 32,000 (640) at 8 5.0 (5.1), at 128
// 17.2 (17.5), at 383 39.5 (43.8); delay of one step.  The launches spread it over the device: 8,000 neurons 10.1 and
// 11.8 (9.6, 10.2), 16,000 9.3 and 10.5 (9.3, 10.2), 32,000 (tiled) 10.9, 12.3 and 13.9 (10.5,
// 11.5, 13.7).
double degree_of(const snn_network *net) { return net->n ? (double)net->nnz / net->n : 0.0; }
double solo_us(const snn_network *net, double spikes) {
  return 0.9 + 0.105e-3 * net->n + spikes * (0.02 + 0.13e-3 * degree_of(net));
}
double launches_us(const snn_network *net, double spikes) {
  const double events = spikes * degree_of(net) * net->window;
  const double window = net->delivery == SNN_DELIVERY_TILED
                            ? 10.4 + 0.0135e-3 * events
                            : std::min(7.6 + 0.04e-3 * net->n, 6.4 + 0.3e-3 * net->n) + 0.033e-3 * events;
  return window / net->window;
}

// Whether a rate in use makes the launches the faster way, so that the rate has to be known.
// (Networks of up to some 8,000 neurons with rows of 80 are persistent at any such rate.)
bool rate_matters(const snn_network *net) {
  return net->solo && solo_us(net, spikes_at(net, kHighHz)) > launches_us(net, spikes_at(net, kHighHz));
}

// Spikes per step that the persistent kernel's launches are sized for.
double expected_spikes(const snn_network *net) {
  return net->spikes_per_step >= 0.0 ? net->spikes_per_step : spikes_at(net, kHighHz);
}

// Steps for which the persistent kernel serves whatever the rate: enough for what a program runs
// before it first looks, some milliseconds where the launches were the faster way (32,000
// neurons with 640 synapses each at 40 Hz: 3.4 ms lost, at 3 Hz 2.6 ms gained).
constexpr uint64_t kGuessSteps = 512;

// Whether snn_run takes the persistent kernel now.  Before the rate is known, and after the first
// steps, it does where that loses less at 100 Hz than the launches lose at 15 Hz: by this model
// 20,000 neurons with 400 synapses each 1.5 times against 2.0, 32,000 with 640 2.8 times against
// 1.2.
bool risks_less(const snn_network *net) {
  const double low = spikes_at(net, kLowHz), high = spikes_at(net, kHighHz);
  return solo_us(net, high) / launches_us(net, high) <= launches_us(net, low) / solo_us(net, low);
}
bool solo_now(const snn_network *net) {
  if (!net->solo || !rate_matters(net)) return net->solo;
  if (net->spikes_per_step < 0.0) return net->t_host < kGuessSteps || risks_less(net);
  return solo_us(net, net->spikes_per_step) <= launches_us(net, net->spikes_per_step);
}
// Steps of the persistent kernel until the route is to be looked at again.
uint64_t solo_steps(const snn_network *net, uint64_t n_steps) {
  if (!rate_matters(net) || net->spikes_per_step >= 0.0 || risks_less(net)) return n_steps;
  return std::min(n_steps, kGuessSteps - net->t_host);
}

// Steps a rate is taken over.
constexpr uint64_t kRateSteps = 64, kRateStepsMost = 256;
constexpr uint64_t kRateGapMost = 4096;  // steps until it is looked at again, where it keeps the route

// `count` spikes in the latest `steps` steps, known from a download of them: downloads of few
// steps are added up.
void note_spikes(snn_network *net, uint64_t count, uint64_t steps) {
  if (!rate_matters(net)) return;
  net->noted_spikes += (double)count;
  net->noted_steps += steps;
  if (net->noted_steps < kRateSteps) return;
  net->spikes_per_step = net->noted_spikes / (double)net->noted_steps;
  net->rate_at = net->t_host;
  net->noted_spikes = 0.0;
  net->noted_steps = 0;
}

uint64_t count_spikes(snn_network *net, uint64_t t0, uint64_t t1);

// Counts the spikes of the latest steps where enough have passed since the last count, in a call
// that waits for the device: two launches and a wait, 15 to 25 us.  Counts that confirm the route
// become rarer (a program that waits every 70 steps would pay 6 % of 20,000 neurons' 3.5 us a step
// for one in each wait).
void measure_spikes(snn_network *net) {
  if (!rate_matters(net) || net->t_host - net->rate_at < net->rate_gap) return;
  const bool before = solo_now(net);
  const uint64_t steps = std::min<uint64_t>({net->t_host - net->rate_at, net->raster_cap, kRateStepsMost});
  net->spikes_per_step = (double)count_spikes(net, net->t_host - steps, net->t_host) / (double)steps;
  net->rate_gap = solo_now(net) == before ? std::min(2 * net->rate_gap, kRateGapMost) : kRateSteps;
  net->rate_at = net->t_host;
  net->noted_spikes = 0.0;
  net->noted_steps = 0;
}

// Steps per persistent launch: long enough to amortise the launch and the state's way in
// and out, and of a network by itself no more than an estimated tenth of a second.
constexpr uint32_t kMaxChunk = 1u << 14;
uint64_t solo_chunk(const snn_network *net) {
  return std::min<uint64_t>(kMaxChunk, std::max<uint64_t>(256, (uint64_t)(1e5 / solo_us(net, expected_spikes(net)))));
}

void run_solo(snn_network *net, uint64_t n_steps) {
  const snn::BatchNet d = batch_net(net);
  const snn::LdsPlan lds = lds_plan(solo_need(net), net->n, net->lds_limit - snn::kBatchStaticLds);
  const uint64_t most = solo_chunk(net);
  while (n_steps > 0) {
    const uint32_t chunk = (uint32_t)std::min<uint64_t>(n_steps, most);
    check(snn::launch_solo(d, chunk, snn::kBatchCommit | snn::kBatchWriteRaster | snn::kBatchQueues, lds,
                           net->stream),
          "persistent launch");
    net->t_host += chunk;
    n_steps -= chunk;
  }
}

void dev_free(snn_network *net, void *p);

// ---- windows of an eagerly plastic network -------------------------------------------
// Device memory for the arriving rows of a window as the ranges read them (rows past it are
// read where they are).
constexpr size_t kWindowRowBytes = (size_t)256 << 20;

// Targets of a workgroup: one range per CU while that leaves a wavefront of targets each.
uint32_t window_range(const snn_network *net) {
  const uint32_t share = (net->n + net->cu_count - 1) / net->cu_count;
  return std::min((share + 63) / 64 * 64, snn::kPlasticBlock);
}

// Whether snn_run steps the network in windows (plastic.hip), with the buffers they need: an
// eagerly plastic network with nothing about its delivery chosen by the caller and a delay of
// at least two steps (a window is at most delay - 1 steps).  Two launches per window against
// three per step, in us per step: delay 2 (one-step windows) 11.0 against 12.6 with 500
// neurons, 13.7 against 19.3 with 20,000, 20.4 against 22.5 with 60,000; delay 10, 3.9 against
// 19.3 with 20,000; delay 15, 2.6 against 14.0 with 4,000 and 9.1 against 22.7 with 60,000.
// Every range looks at every arriving spike, so rows of fewer synapses than half the ranges
// stay with the launches (200,000 neurons with 500 synapses each, 1.3 per range: 24.7 against
// 40.8), and so does a network whose memory has no room for the windows' index.
bool choose_windows(snn_network *net) {
  if (!net->plastic || net->lazy || net->owner || net->delay < 2 || net->n == 0 || net->delivery_chosen ||
      net->prm.window)
    return false;
  const uint32_t range = window_range(net), ranges = (net->n + range - 1) / range;
  if ((double)net->nnz < 0.5 * (double)ranges * net->n) return false;
  if (net->range_off) return true;
  const bool off16 = net->row_len_bound < 65536;
  const size_t entries = (size_t)net->n * (ranges + 1);
  // Lanes of a sub-row (their lengths are about Poisson): nearly every one fits.  A workgroup has
  // kPlasticAhead of them per lane group in flight and takes what is beyond one by one, which at
  // twice as many spikes a step is slower than the launches; where a rate in use brings that
  // many, the lanes go down to the mean and a deviation.  100,000 neurons with 2,000 synapses each (8.9
  // a sub-row), at 852 / 500 / 148 spikes a step: 32 lanes 129 / 68.9 / 18.8 us, 16 lanes 94 / 49.4 /
  // 17.0 (launches 103 / 59.8 / 33.8); 60,000 (5.1) at 937 / 743: 16 lanes 76.5 / 63.8, 8 lanes 55.1 / 47.2
  // (69.5 / 62.8); 300,000 (1.5) at 3,316 / 772: 8 lanes 268 / 64.7, 4 lanes 203 / 53.3 (215 / 66.8).  At
  // low rates the long sub-rows cost more than is gained (10,000 neurons, 1.3 a sub-row: 3.8 us with 8
  // lanes, 4.0 with 4).
  const double mean = (double)net->nnz / ((double)net->n * ranges), rows = spikes_at(net, kHighHz);
  uint32_t shift = lanes_shift_for(mean + 2.5 * std::sqrt(mean) + 0.5, 1);
  const uint32_t fewest = lanes_shift_for(mean + std::sqrt(mean) + 0.5, 1);
  while (shift > fewest && rows > 2.0 * (snn::kPlasticAhead * snn::kPlasticBlock >> shift)) --shift;
  const size_t row_bytes = (size_t)ranges * (sizeof(snn::SubRow) + (sizeof(uint16_t) << shift));
  const uint32_t cap = (uint32_t)std::min<size_t>(snn::kPlasticRows, kWindowRowBytes / row_bytes);
  const uint32_t slots = net->delay + std::min(net->delay - 1, snn::kPlasticSteps) + 1;
  void *held[7] = {};
  try {
    held[0] = off16 ? (void *)dev_array<uint16_t>(net, entries) : (void *)dev_array<uint32_t>(net, entries);
    held[1] = dev_array<uint2>(net, 2 * (size_t)net->n);
    held[2] = dev_array<uint4>(net, 2 * (size_t)net->n);
    held[3] = dev_array<int32_t>(net, (size_t)slots * net->n);
    held[4] = dev_array<uint32_t>(net, (size_t)(slots + 3) * snn::kQlenStride);
    held[5] = dev_array<snn::SubRow>(net, (size_t)std::max(cap, 1u) * ranges);
    held[6] = dev_array<uint16_t>(net, ((size_t)std::max(cap, 1u) * ranges) << shift);
  } catch (...) {
    for (void *p : held)
      if (p) dev_free(net, p);
    return false;
  }
  check(snn::launch_tile_index(net->row_ptr, net->col, net->n, net->nnz, net->nnz, ranges, range, nullptr, held[0],
                               off16, net->stream),
        "range index");
  net->range_off = held[0];
  net->trace = static_cast<uint2 *>(held[1]);
  net->ltp = static_cast<uint4 *>(held[2]);
  net->spike_list = static_cast<int32_t *>(held[3]);
  net->spike_list_len = static_cast<uint32_t *>(held[4]);
  net->row_head = static_cast<snn::SubRow *>(held[5]);
  net->row_tgt = static_cast<uint16_t *>(held[6]);
  net->list_slots = slots;
  net->row_cap = cap;
  net->row_shift = shift;
  net->range = range;
  net->ranges = ranges;
  return true;
}

snn::PlasticArgs plastic_args(snn_network *net) {
  snn::PlasticArgs a{};
  a.row_ptr = net->row_ptr;
  a.col = net->col;
  a.w_f32 = net->w_f32;
  a.plast_rel = net->plast_rel;
  a.plast_len = net->plast_len;
  a.in_ptr = net->in_ptr;
  a.in_src = net->in_src;
  a.in_edge = net->in_edge;
  a.off = net->range_off;
  for (uint32_t k = 0; k < 2; ++k) {
    a.trace[k] = net->trace + (size_t)k * net->n;
    a.ltp[k] = net->ltp + (size_t)k * net->n;
    a.ltp_len[k] = net->spike_list_len + (size_t)(net->list_slots + k) * snn::kQlenStride;
  }
  a.list = net->spike_list;
  a.list_len = net->spike_list_len;
  a.list_slots = net->list_slots;
  a.arriving = net->spike_list_len + (size_t)(net->list_slots + 2) * snn::kQlenStride;
  a.row_head = net->row_head;
  a.row_tgt = net->row_tgt;
  a.row_cap = net->row_cap;
  a.row_blocks = std::min(net->cu_count * 4, std::max(64u, net->n / 64));
  a.v = net->v;
  a.ref = net->ref;
  a.input = net->input;
  a.x_pre = net->x_pre;
  a.x_post = net->x_post;
  a.q = queue_ref(net);
  a.raster = net->raster;
  a.table32 = net->d_table32;
  a.guide = net->d_guide;
  a.ctl = net->ctl;
  a.n = net->n;
  a.slots = net->slots;
  a.raster_cap = net->raster_cap;
  a.words = net->words;
  a.table_len = net->table_len;
  a.delay = net->delay;
  a.range = net->range;
  a.ranges = net->ranges;
  a.off16 = net->row_len_bound < 65536 ? 1u : 0u;
  a.lanes_shift = net->row_shift;
  a.key0 = net->key0;
  a.key1 = net->key1;
  a.alpha = net->alpha;
  a.v_inf = net->v_inf;
  a.v_th = net->v_th;
  a.v_reset = net->v_reset;
  a.beta_plus = net->beta_plus;
  a.beta_minus = net->beta_minus;
  a.ref_steps = net->ref_steps;
  a.w_ext_q16 = net->w_ext_q16;
  a.a_plus = net->a_plus;
  a.a_minus = net->a_minus;
  a.w_max = net->w_max;
  return a;
}

void run_windows(snn_network *net, uint64_t n_steps) {
  snn::PlasticArgs a = plastic_args(net);
  check(snn::launch_plastic_import(a, net->stream), "spike lists");
  const uint32_t most = std::min(net->delay - 1, snn::kPlasticSteps);
  for (bool first = true; n_steps > 0; first = false) {
    const uint32_t steps = (uint32_t)std::min<uint64_t>(n_steps, most);
    a.first = first;
    a.last = steps == n_steps;
    a.ltp_blocks = first ? 0u : std::min(net->cu_count * 8, std::max(64u, net->n / 32));
    check(snn::launch_plastic_window(a, steps, net->stream), "plastic window");
    a.parity ^= 1u;
    net->t_host += steps;
    n_steps -= steps;
  }
  a.ltp_blocks = std::min(net->cu_count * 8, std::max(64u, net->n / 32));
  check(snn::launch_plastic_export(a, net->stream), "potentiation and spike queues");
}

void ensure_graph(snn_network *net) {
  if (net->graph) return;
  const uint32_t windows = std::max(1u, (64u + net->window - 1) / net->window);
  const uint32_t steps = windows * net->window;
  hipGraph_t g = nullptr;
  check(hipStreamBeginCapture(net->stream, hipStreamCaptureModeRelaxed), "begin capture");
  const uint64_t saved = net->t_host;
  try {
    for (uint32_t k = 0; k < windows; ++k) issue_window(net, net->window);
  } catch (...) {
    (void)hipStreamEndCapture(net->stream, &g);
    if (g) (void)hipGraphDestroy(g);
    net->t_host = saved;
    throw;
  }
  net->t_host = saved;
  check(hipStreamEndCapture(net->stream, &g), "end capture");
  const hipError_t e = hipGraphInstantiate(&net->graph, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  check(e, "graph instantiate");
  net->graph_steps = steps;
}

// How a run of more than one step goes (the windows after the launches that queues written by
// the caller still need).
uint32_t route(const snn_network *net) {
  if (net->profiling) return SNN_ROUTE_LAUNCHES;
  return solo_now(net) ? SNN_ROUTE_PERSISTENT : net->windows ? SNN_ROUTE_WINDOWS : SNN_ROUTE_LAUNCHES;
}

void run(snn_network *net, uint64_t n_steps) {
  if (n_steps > 1 && route(net) == SNN_ROUTE_PERSISTENT) {
    const uint64_t steps = solo_steps(net, n_steps);
    run_solo(net, steps);
    n_steps -= steps;
  }
  const uint32_t way = n_steps > 1 ? route(net) : SNN_ROUTE_LAUNCHES;
  if (way == SNN_ROUTE_WINDOWS) {
    for (; n_steps > 0 && net->t_host < net->windows_from; --n_steps) issue_window(net, 1);
    if (n_steps > 0) run_windows(net, n_steps);
    return;
  }
  while (n_steps > 0) {
    // (capturing a graph takes the host as long as some ten windows: a short first run, with
    // which a network may also end, is launched directly)
    if (!net->profiling && n_steps >= 64 && net->stream && (net->graph || net->t_host > 0 || n_steps >= 256)) {
      ensure_graph(net);
      if (n_steps >= net->graph_steps) {
        check(hipGraphLaunch(net->graph, net->stream), "graph launch");
        net->t_host += net->graph_steps;
        n_steps -= net->graph_steps;
        continue;
      }
    }
    const uint32_t steps = (uint32_t)std::min<uint64_t>(n_steps, net->window);
    issue_window(net, steps);
    n_steps -= steps;
  }
}

void sync(snn_network *net) {
  check(hipStreamSynchronize(net->stream), "stream sync");
}

struct CtlTotals {
  uint64_t t, events, spikes, touches, lazy_overrun;
};

CtlTotals sum_ctl(const snn::Ctl &c) {
  CtlTotals r{c.t, 0, 0, 0, c.lazy_overrun};
  for (uint32_t p = 0; p < snn::kCounterParts; ++p) {
    r.events += c.events[p * snn::kLineU64];
    r.spikes += c.spikes[p * snn::kLineU64];
    r.touches += c.touches[p * snn::kLineU64];
  }
  return r;
}

CtlTotals read_ctl(snn_network *net) {
  std::vector<snn::Ctl> c(1);
  check(hipMemcpyAsync(c.data(), net->ctl, sizeof(snn::Ctl), hipMemcpyDeviceToHost, net->stream), "read control");
  sync(net);
  return sum_ctl(c[0]);
}

void raster_range_check(snn_network *net, uint64_t t0, uint64_t t1) {
  if (t1 < t0) fail(SNN_E_INVALID, "t_end < t_begin");
  if (t1 > net->t_host) fail(SNN_E_INVALID, "raster range beyond the simulated steps");
  if (net->t_host - t0 > net->raster_cap) fail(SNN_E_INVALID, "raster range no longer held by the ring");
}

void copy_raster_rows(snn_network *net, uint64_t t0, uint64_t t1, uint64_t *out) {
  const size_t row = (size_t)net->words * 8;
  for (uint64_t t = t0; t < t1;) {
    const uint64_t r = t % net->raster_cap;
    const uint64_t run = std::min<uint64_t>(t1 - t, net->raster_cap - r);
    check(hipMemcpyAsync(out + (t - t0) * net->words, net->raster + r * net->words, run * row,
                         hipMemcpyDeviceToHost, net->stream), "raster copy");
    t += run;
  }
  sync(net);
}


// The download kernels' arguments for steps [t0, t1) (not empty), with `piece` pairs of room in
// the staging behind the count.
constexpr size_t kStageHead = 256;  // the count, on a line of its own
constexpr size_t kPairBytes = 2 * sizeof(uint32_t);
snn::RasterArgs raster_args(snn_network *net, uint64_t t0, uint64_t t1, const Stage &stage, uint64_t piece) {
  snn::RasterArgs a{};
  a.raster = net->raster;
  a.ring_words = (uint64_t)net->raster_cap * net->words;
  a.first_word = t0 % net->raster_cap * net->words;
  a.total_words = (t1 - t0) * net->words;
  a.t_begin = t0;
  a.offset = net->raster_offset;
  a.scratch = net->raster_scratch;
  a.words = net->words;
  a.count = reinterpret_cast<uint64_t *>(stage.data());
  a.steps = reinterpret_cast<uint32_t *>(stage.data() + kStageHead);
  a.ids = a.steps + piece;
  return a;
}

struct Drained {  // a staging block goes back only after nothing writes to it any more
  hipStream_t s;
  ~Drained() { (void)hipStreamSynchronize(s); }
};

// Number of spikes of steps [t0, t1), which the raster holds.
uint64_t count_spikes(snn_network *net, uint64_t t0, uint64_t t1) {
  Stage stage(kStageHead);
  Drained drained{net->stream};
  const snn::RasterArgs a = raster_args(net, t0, t1, stage, 0);
  check(snn::launch_raster_pairs(a, net->stream), "raster count");
  sync(net);
  return *a.count;
}

// The spikes of steps [t0, t1) as sorted pairs in the caller's arrays, their number in
// *n_spikes.  Device kernels find the pairs and write them into pinned staging, in pieces if
// they do not fit one block; the caller's arrays are written only once the count is known
// to fit them.
void download_pairs(snn_network *net, uint64_t t0, uint64_t t1, uint32_t *steps, uint32_t *ids,
                    uint64_t capacity, uint64_t *n_spikes) {
  *n_spikes = 0;
  if (t0 == t1) return;
  // (the clamp keeps the product in range for any capacity)
  Stage stage(kStageHead + std::min<uint64_t>(capacity, kStageMaxBytes / kPairBytes) * kPairBytes);
  Drained drained{net->stream};
  const uint64_t piece = (stage.bytes() - kStageHead) / kPairBytes;
  snn::RasterArgs a = raster_args(net, t0, t1, stage, piece);
  a.out_cap = steps && ids ? std::min(capacity, piece) : 0;
  check(snn::launch_raster_pairs(a, net->stream), "raster pairs");
  sync(net);
  const uint64_t count = *a.count;
  *n_spikes = count;
  if (count > capacity) fail(SNN_E_OVERFLOW, "raster holds " + std::to_string(count) + " spikes");
  if (count && (!steps || !ids)) fail(SNN_E_INVALID, "null output arrays");
  if (t1 == net->t_host && t1 > net->rate_at) note_spikes(net, count, t1 - t0);
  for (uint64_t lo = 0; lo < count; lo += piece) {
    if (lo) {
      a.out_lo = lo;
      check(snn::launch_raster_pairs(a, net->stream), "raster pairs");
      sync(net);
    }
    const size_t part = (size_t)std::min(piece, count - lo);
    std::memcpy(steps + lo, a.steps, part * sizeof(uint32_t));
    std::memcpy(ids + lo, a.ids, part * sizeof(uint32_t));
  }
}

// ---- delivery reconfiguration, timing and autotuning --------------------------------
void dev_free(snn_network *net, void *p) {
  for (size_t k = 0; k < net->allocs.size(); ++k)
    if (net->allocs[k].p == p) {
      if (net->has_alloc) net->alloc.free(p, net->allocs[k].bytes, (void *)net->stream, net->alloc.ctx);
      else pool_free(net->device, p, net->allocs[k].bytes);
      net->device_bytes -= net->allocs[k].bytes;
      net->allocs.erase(net->allocs.begin() + (std::ptrdiff_t)k);
      return;
    }
}

// A new delivery variant / tiling / launch shape, taking effect at the next window (the
// input ring holds exactly the pending arrivals at every window boundary, whichever
// variant filled it).  The new configuration is resolved and its tile index built before
// anything of the old one is released; if any of that fails (an impossible block or
// tiling, device memory, a launch), every field and buffer of the old configuration is
// restored, so the network keeps running as before.  Without `by_caller` the launches' delivery
// changes and nothing else: a route of its own that snn_run takes stays.
void set_delivery(snn_network *net, uint32_t delivery, uint32_t tiles, uint32_t block, uint32_t grid,
                  bool by_caller) {
  if (net->lazy) fail(SNN_E_STATE, "lazy plasticity delivers inside its own kernel; there is no variant to choose");
  if (delivery > SNN_DELIVERY_TILED) fail(SNN_E_INVALID, "unknown delivery variant");
  check(hipStreamSynchronize(net->stream), "sync");
  struct Saved {
    uint32_t p_delivery, p_tiles, p_block, p_grid, delivery, block, tiles, tile_size, grid;
    void *tile_off;
    uint16_t *col16;
    bool tile_off16, solo, windows, chosen;
  };
  const Saved old{net->prm.delivery, net->prm.tiles, net->prm.block, net->prm.grid, net->delivery,
                  net->block,        net->tiles,     net->tile_size, net->grid,     net->tile_off,
                  net->col16,        net->tile_off16, net->solo,     net->windows,   net->delivery_chosen};
  try {
    net->prm.delivery = delivery;
    net->prm.tiles = tiles;
    net->prm.block = block;
    net->prm.grid = grid;
    net->delivery = delivery;
    choose_delivery(net);
    if (net->delivery == SNN_DELIVERY_TILED) {
      net->tile_off = nullptr;  // a fresh index; the old one stays valid until this succeeds
      fill_tile_offsets(net, alloc_tile_offsets(net));  // reuses col16 when it exists (any tiling's)
      check(hipStreamSynchronize(net->stream), "sync after tile offsets");
    } else {
      net->tile_off = nullptr;
    }
    if (by_caller) {
      net->delivery_chosen = delivery != SNN_DELIVERY_AUTO || tiles || block || grid;
      net->solo = choose_solo(net);
      net->windows = choose_windows(net);
      check(hipStreamSynchronize(net->stream), "sync after the new configuration");
    }
  } catch (...) {
    (void)hipStreamSynchronize(net->stream);  // no index launch may still write a block freed here
    if (net->tile_off && net->tile_off != old.tile_off) dev_free(net, net->tile_off);
    if (net->col16 && net->col16 != old.col16) dev_free(net, net->col16);
    net->prm.delivery = old.p_delivery;
    net->prm.tiles = old.p_tiles;
    net->prm.block = old.p_block;
    net->prm.grid = old.p_grid;
    net->delivery = old.delivery;
    net->block = old.block;
    net->tiles = old.tiles;
    net->tile_size = old.tile_size;
    net->grid = old.grid;
    net->solo = old.solo;
    net->windows = old.windows;
    net->delivery_chosen = old.chosen;
    net->tile_off = old.tile_off;
    net->col16 = old.col16;
    net->tile_off16 = old.tile_off16;
    throw;
  }
  if (old.tile_off) dev_free(net, old.tile_off);
  if (net->col16 && net->delivery != SNN_DELIVERY_TILED) {
    dev_free(net, net->col16);
    net->col16 = nullptr;
  }
  if (net->graph) {
    (void)hipGraphExecDestroy(net->graph);
    net->graph = nullptr;
  }
}

// Mean time (ms) of one delivery launch over one window whose step w dequeues
// per_step[w], with scratch queues, accumulators and control block (the network's own
// state is untouched); *events = synaptic events of one launch.
double time_delivery(snn_network *net, const std::vector<std::vector<uint32_t>> &per_step, uint32_t reps,
                     uint64_t *events) {
  const uint32_t steps = (uint32_t)per_step.size();
  if (steps == 0 || steps > net->window) fail(SNN_E_INVALID, "steps exceeds the network's window");
  if (reps == 0) reps = 1;
  hipStream_t s = net->stream;
  // queue slots 0..steps-1, laid out as the update kernel appends: position p of a step
  // goes to sub-queue p mod kQueueGroups at index p / kQueueGroups
  std::vector<int32_t> queue((size_t)steps * net->queue_stride, 0);
  std::vector<uint32_t> qlen((size_t)net->slots * snn::kQueueGroups * snn::kQlenStride, 0u);
  for (uint32_t w = 0; w < steps; ++w) {
    if (per_step[w].size() > net->n) fail(SNN_E_INVALID, "more ids in a step than neurons");
    for (size_t p = 0; p < per_step[w].size(); ++p) {
      const uint32_t id = per_step[w][p];
      if (id >= net->n) fail(SNN_E_INVALID, "id out of range");
      const uint32_t g = (uint32_t)(p % snn::kQueueGroups), pos = (uint32_t)(p / snn::kQueueGroups);
      queue[(size_t)w * net->queue_stride + (size_t)g * net->group_cap + pos] = (int32_t)id;
      qlen[((size_t)w * snn::kQueueGroups + g) * snn::kQlenStride]++;
    }
  }
  std::vector<snn_network::Alloc> mark(net->allocs);
  const uint64_t bytes_before = net->device_bytes;
  double ms_out = 0.0;
  try {
    int32_t *d_queue = dev_array<int32_t>(net, (size_t)net->slots * net->queue_stride);
    uint32_t *d_qlen = dev_array<uint32_t>(net, qlen.size());
    int32_t *input = dev_array<int32_t>(net, (size_t)net->n_inbuf * net->n);
    snn::Ctl *ctl = dev_array<snn::Ctl>(net, 1);
    check(hipMemcpyAsync(d_queue, queue.data(), queue.size() * 4, hipMemcpyHostToDevice, s), "queue");
    check(hipMemcpyAsync(d_qlen, qlen.data(), qlen.size() * 4, hipMemcpyHostToDevice, s), "queue lengths");
    check(hipMemsetAsync(input, 0, (size_t)net->n_inbuf * net->n * 4, s), "clear");
    // slots 0..steps-1 are the queues delivered by a window starting at t0 when
    // t0 + n_inbuf - delay = 0 (mod slots)
    std::vector<snn::Ctl> c0(1);
    std::memset(c0.data(), 0, sizeof(snn::Ctl));
    c0[0].t_deliver = (uint64_t)net->delay - net->n_inbuf;
    check(hipMemcpyAsync(ctl, c0.data(), sizeof(snn::Ctl), hipMemcpyHostToDevice, s), "ctl");
    check(hipStreamSynchronize(s), "sync");
    snn::DeliverArgs d = deliver_args(net);
    d.q = snn::QueueRef{d_queue, d_qlen, net->queue_stride, net->group_cap};
    d.input = input;
    d.ctl = ctl;
    d.advance = 0;
    check(launch_delivery(net, d, steps), "warm-up delivery");
    // each launch stamped with its own begin and end (no marker packets between them)
    std::vector<snn::LaunchEvents> evs(reps);
    for (auto &e : evs) {
      e.start = pooled_event(net);
      e.stop = pooled_event(net);
    }
    for (uint32_t r = 0; r < reps; ++r) check(launch_delivery(net, d, steps, evs[r]), "delivery");
    check(hipStreamSynchronize(s), "sync");
    float ms = 0.f;
    for (auto &e : evs) {
      float one = 0.f;
      check(hipEventElapsedTime(&one, e.start, e.stop), "elapsed");
      ms += one;
      net->event_pool.push_back(e.start);
      net->event_pool.push_back(e.stop);
    }
    std::vector<snn::Ctl> c1(1);
    check(hipMemcpy(c1.data(), ctl, sizeof(snn::Ctl), hipMemcpyDeviceToHost), "ctl");
    ms_out = ms / reps;
    if (events) *events = sum_ctl(c1[0]).events / (reps + 1);
  } catch (...) {
    (void)hipStreamSynchronize(s);  // no launch may still use the scratch handed back below
    for (size_t k = mark.size(); k < net->allocs.size(); ++k) {
      if (net->has_alloc) net->alloc.free(net->allocs[k].p, net->allocs[k].bytes, (void *)s, net->alloc.ctx);
      else pool_free(net->device, net->allocs[k].p, net->allocs[k].bytes);
    }
    net->allocs.resize(mark.size());
    net->device_bytes = bytes_before;
    throw;
  }
  for (size_t k = mark.size(); k < net->allocs.size(); ++k) {
    if (net->has_alloc) net->alloc.free(net->allocs[k].p, net->allocs[k].bytes, (void *)s, net->alloc.ctx);
    else pool_free(net->device, net->allocs[k].p, net->allocs[k].bytes);
  }
  net->allocs.resize(mark.size());
  net->device_bytes = bytes_before;
  return ms_out;
}

// ---- delivery timing in a fixed device array (no allocation) ------------------------
// Scratch of snn_time_delivery_static: one window's staged queues and counters, the
// control block and the input accumulators the delivery writes.  Each GPU holds its
// own copy for the life of the process; host code reaches it only through the address
// hipGetSymbolAddress returns for that device.
constexpr size_t kStaticScratchBytes = 64ull << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
struct StaticScratch {
  unsigned char *ptr = nullptr;            // device address of `scratch` on this device
  hipEvent_t start = nullptr, stop = nullptr;  // timing events, created with it
};
std::mutex g_static_mu;
StaticScratch g_static[kMaxDevices];

// Set-up on the first call on `device`, with that device current: the array's device
// address and the two timing events.  Later calls only read the table.
StaticScratch static_scratch(int device) {
  if (device < 0 || device >= kMaxDevices) fail(SNN_E_INVALID, "device id beyond the static scratch table");
  std::lock_guard<std::mutex> lock(g_static_mu);
  StaticScratch &s = g_static[device];
  if (s.ptr) return s;
  int cur = -1;
  check(hipGetDevice(&cur), "hipGetDevice");
  if (cur != device) check(hipSetDevice(device), "hipSetDevice");
  void *p = nullptr;
  hipEvent_t a = nullptr, b = nullptr;
  hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e == hipSuccess) e = hipEventCreate(&a);
  if (e == hipSuccess) e = hipEventCreate(&b);
  if (cur != device) (void)hipSetDevice(cur);
  if (e != hipSuccess || !p) {
    if (a) (void)hipEventDestroy(a);
    if (b) (void)hipEventDestroy(b);
    check(e != hipSuccess ? e : hipErrorInvalidSymbol, "static scratch set-up");
  }
  s.start = a;
  s.stop = b;
  s.ptr = static_cast<unsigned char *>(p);
  return s;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// snn_time_delivery with every device buffer in the static scratch: the ids are checked
// on the host, copied into the scratch as they are, and laid out as the window's queues
// by k_stage_window; then one untimed and `reps` timed launches of the network's
// delivery kernel, the mean taken from the first timed launch's begin to the last one's
// end.
double time_delivery_static(snn_network *net, const uint32_t *ids, uint32_t n_ids, const uint32_t *step_counts,
                            uint32_t steps, uint32_t reps, uint64_t *events) {
  if (steps == 0 || steps > net->window) fail(SNN_E_INVALID, "steps exceeds the network's window");
  if (reps == 0) reps = 1;
  snn::StageArgs st{};
  st.steps = steps;
  st.n_ids = n_ids;
  st.round_robin = step_counts ? 0u : 1u;
  uint64_t k = 0;
  for (uint32_t w = 0; w < steps; ++w) {
    const uint64_t c = step_counts ? step_counts[w] : (n_ids > w ? (n_ids - w + steps - 1) / steps : 0u);
    if (c > net->n) fail(SNN_E_INVALID, "more ids in a step than neurons");
    st.off[w] = (uint32_t)k;
    k += c;
    if (k > n_ids) fail(SNN_E_INVALID, "step counts exceed the ids");
  }
  if (k != n_ids) fail(SNN_E_INVALID, "step counts do not sum to n_ids");
  st.off[steps] = (uint32_t)k;
  for (uint32_t j = 0; j < n_ids; ++j)
    if (ids[j] >= net->n) fail(SNN_E_INVALID, "id out of range");
  const size_t o_qlen = align256(sizeof(snn::Ctl));
  const size_t o_queue = o_qlen + align256((size_t)steps * snn::kQueueGroups * snn::kQlenStride * 4);
  const size_t o_input = o_queue + align256((size_t)steps * net->queue_stride * 4);
  const size_t o_ids = o_input + align256((size_t)net->n_inbuf * net->n * 4);
  const size_t need = o_ids + align256((size_t)n_ids * 4);
  if (need > kStaticScratchBytes)
    fail(SNN_E_INVALID, "this window needs " + std::to_string(need) + " bytes of device scratch; the static scratch holds " +
                            std::to_string(kStaticScratchBytes));
  const StaticScratch sc = static_scratch(net->device);
  hipStream_t s = net->stream;
  snn::Ctl *ctl = reinterpret_cast<snn::Ctl *>(sc.ptr);
  st.q = snn::QueueRef{reinterpret_cast<int32_t *>(sc.ptr + o_queue), reinterpret_cast<uint32_t *>(sc.ptr + o_qlen),
                       net->queue_stride, net->group_cap};
  st.ctl = ctl;
  st.input = reinterpret_cast<int32_t *>(sc.ptr + o_input);
  st.n_input = (uint64_t)net->n_inbuf * net->n;
  st.ids = reinterpret_cast<const int32_t *>(sc.ptr + o_ids);
  // slots 0..steps-1 are the queues delivered by a window starting at t0 when
  // t0 + n_inbuf - delay = 0 (mod slots)
  st.t_deliver = (uint64_t)net->delay - net->n_inbuf;
  if (n_ids)
    check(hipMemcpyAsync(sc.ptr + o_ids, ids, (size_t)n_ids * 4, hipMemcpyHostToDevice, s), "ids");
  check(snn::launch_stage_window(st, s), "stage window");
  snn::DeliverArgs d = deliver_args(net);
  d.q = st.q;
  d.input = st.input;
  d.ctl = ctl;
  d.advance = 0;
  check(launch_delivery(net, d, steps), "warm-up delivery");
  for (uint32_t r = 0; r < reps; ++r) {
    snn::LaunchEvents ev;
    if (r == 0) ev.start = sc.start;
    if (r + 1 == reps) ev.stop = sc.stop;
    check(launch_delivery(net, d, steps, ev), "delivery");
  }
  uint64_t parts[snn::kCounterParts];
  check(hipMemcpy2DAsync(parts, sizeof(uint64_t), ctl->events, snn::kLineU64 * sizeof(uint64_t), sizeof(uint64_t),
                         snn::kCounterParts, hipMemcpyDeviceToHost, s),
        "event counters");
  check(hipStreamSynchronize(s), "sync");
  float ms = 0.f;
  check(hipEventElapsedTime(&ms, sc.start, sc.stop), "elapsed");
  uint64_t total = 0;
  for (uint64_t x : parts) total += x;
  if (events) *events = total / (reps + 1);
  return (double)ms / reps;
}

// Times every candidate delivery configuration on the spikes of the latest window (read
// from the raster ring) and keeps the fastest for the launches.  The tuner's choice is not the
// caller's: a network that snn_run advances by a route of its own (which delivers inside its own
// kernels) keeps it.  (With the choice taken for the caller's, a tuned 4,000-neuron network went
// from 1.4 to 8 us per step and a plastic one of 10,000 from 3 to 16.)
snn_delivery_tuning autotune_delivery(snn_network *net, uint32_t reps) {
  if (net->lazy) fail(SNN_E_STATE, "lazy plasticity delivers inside its own kernel; there is no variant to tune");
  const uint32_t W = net->window;
  if (net->t_host < W) fail(SNN_E_STATE, "run at least one window before autotuning the delivery");
  if (net->raster_cap < W) fail(SNN_E_STATE, "the raster ring holds less than one window");
  sync(net);
  std::vector<uint64_t> rows((size_t)W * net->words);
  raster_range_check(net, net->t_host - W, net->t_host);
  copy_raster_rows(net, net->t_host - W, net->t_host, rows.data());
  std::vector<std::vector<uint32_t>> per_step(W);
  for (uint32_t w = 0; w < W; ++w)
    for (uint32_t k = 0; k < net->words; ++k) {
      uint64_t m = rows[(size_t)w * net->words + k];
      while (m) {
        const uint32_t b = (uint32_t)__builtin_ctzll(m);
        m &= m - 1;
        per_step[w].push_back(k * 64 + b);
      }
    }
  struct Cand {
    uint32_t delivery, tiles, block, grid;
  };
  std::vector<Cand> cands;
  cands.push_back({SNN_DELIVERY_ATOMIC, 0, 0, 0});
  if (net->n >= 1024) {
    for (uint32_t tile : {384u, 576u, 768u})
      for (uint32_t block : {512u, 1024u})
        for (uint32_t grid : {net->cu_count, 2 * net->cu_count, 3 * net->cu_count})
          cands.push_back({SNN_DELIVERY_TILED, std::max(1u, (net->n + tile - 1) / tile), block, grid});
  }
  const Cand keep{net->prm.delivery, net->prm.tiles, net->prm.block, net->prm.grid};
  snn_delivery_tuning best{};
  best.ms_per_launch = 1e300;
  try {
    for (const Cand &c : cands) {
      try {
        set_delivery(net, c.delivery, c.tiles, c.block, c.grid, false);
      } catch (const Failure &) {
        continue;  // e.g. a tile larger than the LDS allows
      }
      uint64_t ev = 0;
      const double ms = time_delivery(net, per_step, reps, &ev);
      if (ms < best.ms_per_launch) {
        best.ms_per_launch = ms;
        best.delivery = net->delivery;
        best.tiles = net->tiles;
        best.block = net->block;
        best.grid = net->grid;
        best.events_per_launch = ev;
      }
    }
    if (best.ms_per_launch == 1e300) fail(SNN_E_STATE, "no delivery configuration could be timed");
    set_delivery(net, best.delivery, best.tiles, best.block, best.grid, false);
  } catch (...) {
    try {
      set_delivery(net, keep.delivery, keep.tiles, keep.block, keep.grid, false);
    } catch (...) {
    }
    throw;
  }
  return best;
}

// ---- batched form ----------------------------------------------------------------
}  // namespace

struct snn_batch {
  std::vector<snn_network *> nets;
  snn_network pool;                  // holds the batch's own allocations and stream
  std::vector<snn::BatchNet> desc;
  std::vector<double> degree;        // mean out-degree of each member
  std::vector<uint32_t> order;       // workgroup -> member, heaviest first
  snn::BatchNet *d_desc = nullptr;
  uint32_t *d_order = nullptr;
  uint32_t n_max = 0;
  size_t lds_need = 0;               // dynamic LDS of the largest member
  uint32_t lds_limit = 0;
  size_t lds_budget = 0;             // dynamic LDS a launch may use
  snn_batch_tuning tuning{};
  std::vector<std::pair<uint32_t, hipGraphExec_t>> graphs;  // by steps per launch
};

namespace {

void batch_clear_graphs(snn_batch *b) {
  for (auto &g : b->graphs) (void)hipGraphExecDestroy(g.second);
  b->graphs.clear();
}

void batch_apply_tuning(snn_batch *b, const snn_batch_tuning &t) {
  if (t.block != 256 && t.block != 512 && t.block != 1024) fail(SNN_E_INVALID, "block must be 256, 512 or 1024");
  if (t.degree_div != 1 && t.degree_div != 2 && t.degree_div != 4 && t.degree_div != 8 && t.degree_div != 16)
    fail(SNN_E_INVALID, "degree_div must be 1, 2, 4, 8 or 16");
  const uint32_t per = snn::batch_per_lane(t.block, b->n_max);
  if (per == 0) fail(SNN_E_INVALID, "largest network does not fit a workgroup of this size");
  for (size_t k = 0; k < b->desc.size(); ++k) b->desc[k].lanes_shift = lanes_shift_for(b->degree[k], t.degree_div);
  check(hipMemcpyAsync(b->d_desc, b->desc.data(), b->desc.size() * sizeof(snn::BatchNet), hipMemcpyHostToDevice,
                       b->pool.stream), "copy batch descriptors");
  check(hipStreamSynchronize(b->pool.stream), "sync");
  b->tuning = t;
  b->tuning.per_lane = per;
  b->tuning.pad_ = 0;
  batch_clear_graphs(b);
}

void batch_launch(snn_batch *b, uint32_t steps, uint32_t flags) {
  for (const snn::BatchNet &d : b->desc)
    if (d.below) flags |= snn::kBatchDrive;
  const snn::LdsPlan lds = lds_plan(b->lds_need, b->n_max, b->lds_budget);
  check(snn::launch_batch(b->d_desc, b->d_order, (uint32_t)b->nets.size(), steps, b->tuning.block,
                          b->tuning.per_lane, flags, lds, b->pool.stream), "batch launch");
}

hipGraphExec_t batch_graph(snn_batch *b, uint32_t steps) {
  for (auto &g : b->graphs)
    if (g.first == steps) return g.second;
  hipGraph_t g = nullptr;
  hipStream_t s = b->pool.stream;
  check(hipStreamBeginCapture(s, hipStreamCaptureModeRelaxed), "begin capture");
  try {
    batch_launch(b, steps, snn::kBatchCommit | snn::kBatchWriteRaster);
  } catch (...) {
    (void)hipStreamEndCapture(s, &g);
    if (g) (void)hipGraphDestroy(g);
    throw;
  }
  check(hipStreamEndCapture(s, &g), "end capture");
  hipGraphExec_t ex = nullptr;
  const hipError_t e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  check(e, "graph instantiate");
  if (b->graphs.size() >= 8) batch_clear_graphs(b);
  b->graphs.push_back({steps, ex});
  return ex;
}

// Each launch advances every member by `chunk` steps; one kernel node per launch,
// replayed from a graph captured once per chunk length.
void batch_run(snn_batch *b, uint64_t n_steps) {
  while (n_steps > 0) {
    const uint32_t chunk = (uint32_t)std::min<uint64_t>(n_steps, kMaxChunk);
    check(hipGraphLaunch(batch_graph(b, chunk), b->pool.stream), "graph launch");
    for (snn_network *m : b->nets) m->t_host += chunk;
    n_steps -= chunk;
  }
}

void batch_destroy(snn_batch *b) {
  if (b->pool.stream) (void)hipStreamSynchronize(b->pool.stream);
  batch_clear_graphs(b);
  for (snn_network *m : b->nets) {
    m->owner = nullptr;
    m->own_stream = false;  // the stream belongs to the pool
    release(m);
    delete m;
  }
  b->nets.clear();
  release(&b->pool);
}

void build_batch(snn_batch *b, const snn_batch_member *members, uint32_t n_nets, uint32_t raster_steps) {
  hipStream_t s = b->pool.stream;
  int lds_max = 0;
  check(hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, b->pool.device),
        "LDS limit");
  b->lds_limit = (uint32_t)std::max(0, lds_max - (int)snn::kBatchStaticLds);
  for (uint32_t k = 0; k < n_nets; ++k) {
    const snn_batch_member &mb = members[k];
    if (!mb.params || (!mb.pops && mb.n_pops) || (!mb.proj && mb.n_proj))
      fail(SNN_E_INVALID, "member " + std::to_string(k) + ": null argument");
    snn_network *m = new snn_network();
    b->nets.push_back(m);
    m->owner = b;
    m->prm = *mb.params;
    m->prm.raster_steps = raster_steps;
    m->prm.window = 0;
    m->prm.delivery = SNN_DELIVERY_ATOMIC;
    m->prm.tiles = m->prm.block = m->prm.grid = 0;
    m->pops.assign(mb.pops, mb.pops + mb.n_pops);
    m->proj.assign(mb.proj, mb.proj + mb.n_proj);
    m->alloc = b->pool.alloc;
    m->has_alloc = b->pool.has_alloc;
    m->device = b->pool.device;
    m->cu_count = b->pool.cu_count;
    m->stream = s;
    try {
      build(m);
    } catch (const Failure &f) {
      fail(f.code, "member " + std::to_string(k) + ": " + f.msg);
    }
    if (m->plastic) fail(SNN_E_INVALID, "member " + std::to_string(k) + ": the batched form needs static weights");
    if (m->n_inbuf != m->delay) fail(SNN_E_INVALID, "member " + std::to_string(k) + ": unexpected input ring");
    const uint32_t below = drive_thresholds(m);
    const size_t lds = ((size_t)m->delay * m->n + below) * 4;
    if (m->n > 20480 || lds > b->lds_limit)
      fail(SNN_E_INVALID, "member " + std::to_string(k) + " does not fit one workgroup (n = " + std::to_string(m->n) +
                              ", delay ring + drive table = " + std::to_string(lds) + " bytes of LDS, limit " +
                              std::to_string(b->lds_limit) + ")");
    b->lds_need = std::max(b->lds_need, (lds + 15) & ~(size_t)15);
    b->n_max = std::max(b->n_max, m->n);
    const snn::BatchNet d = batch_net(m);
    b->desc.push_back(d);
    b->degree.push_back(m->n ? (double)m->nnz / m->n : 0.0);
  }
  // Batches of more networks than compute units keep what LDS use lets two or more
  // workgroups share a unit; the others may use all of it.
  b->lds_budget = b->lds_limit;
  if (n_nets > b->pool.cu_count && b->lds_need)
    b->lds_budget = std::max(b->lds_need, (size_t)lds_max / ((size_t)lds_max / (b->lds_need + snn::kBatchStaticLds)) -
                                              snn::kBatchStaticLds);
  // heaviest networks first: the first workgroups start first and get a CU each
  std::vector<double> work(n_nets);
  for (uint32_t k = 0; k < n_nets; ++k) work[k] = (double)b->nets[k]->nnz + 8.0 * b->nets[k]->n;
  b->order.resize(n_nets);
  std::iota(b->order.begin(), b->order.end(), 0u);
  std::stable_sort(b->order.begin(), b->order.end(), [&](uint32_t x, uint32_t y) { return work[x] > work[y]; });
  b->d_desc = dev_array<snn::BatchNet>(&b->pool, std::max<size_t>(1, n_nets));
  b->d_order = dev_array<uint32_t>(&b->pool, std::max<size_t>(1, n_nets));
  check(hipMemcpyAsync(b->d_order, b->order.data(), n_nets * 4, hipMemcpyHostToDevice, s), "copy order");
  snn_batch_tuning t{};
  t.degree_div = 4;
  t.block = 256;
  // 1,024 threads: 3.5 us per step of 96 networks of 1,000 to 20,000 neurons (4.3 with 512,
  // 6.2 with 256), 5.2 of 512 such networks (6.0, 7.4), 1.9 of 64 of up to 5,000 (2.1, 2.5)
  for (uint32_t blk : {1024u, 512u, 256u})
    if (snn::batch_per_lane(blk, b->n_max)) {
      t.block = blk;
      break;
    }
  batch_apply_tuning(b, t);
}

snn_batch_tuning batch_autotune(snn_batch *b, uint32_t trial_steps) {
  if (trial_steps == 0) fail(SNN_E_INVALID, "trial_steps must be positive");
  hipStream_t s = b->pool.stream;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  check(hipEventCreate(&e0), "event");
  check(hipEventCreate(&e1), "event");
  snn_batch_tuning best{};
  double best_ms = 1e300;
  try {
    for (uint32_t blk : {256u, 512u, 1024u}) {
      if (!snn::batch_per_lane(blk, b->n_max)) continue;
      for (uint32_t div : {1u, 2u, 4u, 8u, 16u}) {
        snn_batch_tuning t{};
        t.block = blk;
        t.degree_div = div;
        batch_apply_tuning(b, t);
        batch_launch(b, trial_steps, 0u);  // warm-up
        check(hipEventRecord(e0, s), "event record");
        batch_launch(b, trial_steps, 0u);
        check(hipEventRecord(e1, s), "event record");
        check(hipEventSynchronize(e1), "event sync");
        float ms = 0.f;
        check(hipEventElapsedTime(&ms, e0, e1), "elapsed");
        if (ms < best_ms) {
          best_ms = ms;
          best = b->tuning;
        }
      }
    }
  } catch (...) {
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    throw;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  batch_apply_tuning(b, best);
  b->tuning.ms_per_step = best_ms / trial_steps;
  return b->tuning;
}


// ---- surrogate-gradient BPTT plan ------------------------------------------------
}  // namespace

struct snn_bptt {
  snn_bptt_desc desc{};
  snn_network pool;          // holds the plan's allocations and default stream
  snn::BpttArgs args{};
  uint64_t forwards = 0;     // forward passes run (the backward uses the latest)
  hipGraphExec_t g_fwd = nullptr, g_bwd = nullptr;  // captured bodies of the two passes
  volatile uint32_t *activity = nullptr;  // of a finished pass (BpttArgs::act_out)
  ~snn_bptt() {
    if (activity) slot_give(const_cast<uint32_t *>(activity));
  }
};

namespace {

// Transposed index of a CSR matrix with `rows` rows and `cols` columns: for each
// column, its (row, edge) pairs in ascending row order (a counting sort over rows).
void transpose_csr(const uint64_t *ptr, const int32_t *col, uint32_t rows, uint32_t cols,
                   std::vector<uint64_t> &t_ptr, std::vector<int32_t> &t_src, std::vector<uint32_t> &t_edge) {
  const uint64_t nnz = ptr[rows];
  t_ptr.assign((size_t)cols + 1, 0);
  for (uint64_t e = 0; e < nnz; ++e) t_ptr[(size_t)col[e] + 1]++;
  for (uint32_t c = 0; c < cols; ++c) t_ptr[c + 1] += t_ptr[c];
  std::vector<uint64_t> fill(t_ptr.begin(), t_ptr.end() - 1);
  t_src.assign(nnz ? nnz : 1, 0);
  t_edge.assign(nnz ? nnz : 1, 0);
  for (uint32_t r = 0; r < rows; ++r)
    for (uint64_t e = ptr[r]; e < ptr[r + 1]; ++e) {
      const uint64_t at = fill[(size_t)col[e]]++;
      t_src[at] = (int32_t)r;
      t_edge[at] = (uint32_t)e;
    }
}

void check_csr(const uint64_t *ptr, const int32_t *col, uint32_t rows, uint32_t cols, uint64_t nnz,
               const char *what) {
  if (!ptr || (!col && nnz)) fail(SNN_E_INVALID, std::string(what) + ": null CSR array");
  if (ptr[0] != 0 || ptr[rows] != nnz) fail(SNN_E_INVALID, std::string(what) + ": row pointers do not span nnz");
  if (nnz >= (1ull << 32)) fail(SNN_E_INVALID, std::string(what) + ": more than 2^32 - 1 synapses");
  for (uint32_t r = 0; r < rows; ++r) {
    if (ptr[r + 1] < ptr[r]) fail(SNN_E_INVALID, std::string(what) + ": decreasing row pointers");
    for (uint64_t e = ptr[r]; e < ptr[r + 1]; ++e) {
      if (col[e] < 0 || (uint32_t)col[e] >= cols) fail(SNN_E_INVALID, std::string(what) + ": target out of range");
      if (e > ptr[r] && col[e] <= col[e - 1]) fail(SNN_E_INVALID, std::string(what) + ": row not strictly ascending");
    }
  }
}

template <typename T>
T *upload(snn_network *pool, const std::vector<T> &v) {
  T *d = dev_array<T>(pool, std::max<size_t>(1, v.size()));
  if (!v.empty())
    check(hipMemcpyAsync(d, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, pool->stream), "upload");
  return d;
}

// Deals the rows of W_rec to the lanes of the one-workgroup membrane adjoint and orders every
// lane's synapses (snn_internal.h, seq_*).  Leaves seq_threads 0 where the form does not fit.
//  * `p` neighbouring lanes share a row, the largest power of two (<= 16) with p H <= 1,024;
//    rows go to lanes by descending length, so that a wavefront's rows are about equally long.
//  * A row's synapses are dealt place by place: at each place, every lane takes, among the next
//    few it has left, the one whose LDS bank is least used by the 32 lanes read together.
void build_seq(snn_bptt *pl, const uint64_t *rec_ptr, const int32_t *rec_col) {
  snn::BpttArgs &a = pl->args;
  if (!a.events || !a.S || a.H > snn::kSeqMaxNeurons) return;
  uint32_t p = 1;
  while (p < 16 && 2 * p * a.H <= 1024) p *= 2;
  const uint32_t rows_per_wave = 64 / p, n_waves = (a.H + rows_per_wave - 1) / rows_per_wave, n_thr = n_waves * 64;
  std::vector<uint32_t> order(a.H);
  std::iota(order.begin(), order.end(), 0u);
  std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) {
    return rec_ptr[x + 1] - rec_ptr[x] > rec_ptr[y + 1] - rec_ptr[y];
  });
  // a wavefront's places: its longest row over p lanes, in groups of four
  std::vector<uint32_t> groups(16, 0u), more(16, 0u), row(n_thr, 0xFFFFFFFFu);
  uint32_t g_max = 0, more_all = 0;
  for (uint32_t w = 0; w < n_waves; ++w) {
    const uint32_t r0 = order[w * rows_per_wave];
    const uint64_t len = (rec_ptr[r0 + 1] - rec_ptr[r0] + p - 1) / p;
    if (len > snn::kSeqRegs + 4 * snn::kSeqMaxMore) return;
    groups[w] = (uint32_t)((len + 3) / 4);
    g_max = std::max(g_max, groups[w]);
    more[w] = more_all;
    if (groups[w] > snn::kSeqRegs / 4) more_all += groups[w] - snn::kSeqRegs / 4;
  }
  if (more_all > snn::kSeqMaxMore) return;
  g_max = std::max(1u, g_max);
  const size_t places = (size_t)g_max * n_thr * 4;
  std::vector<uint16_t> col(places, (uint16_t)(snn::kSeqMaxNeurons * 4));  // the zero behind the neurons
  std::vector<uint32_t> pos(rec_ptr[a.H]);
  constexpr uint32_t kLook = 16;
  std::vector<std::vector<uint32_t>> left(64);  // of each lane: edges not yet placed
  for (uint32_t w = 0; w < n_waves; ++w) {
    for (uint32_t l = 0; l < 64; ++l) {
      left[l].clear();
      const uint32_t k = w * rows_per_wave + l / p;
      if (k >= a.H) continue;
      row[w * 64 + l] = order[k];
      for (uint64_t e = rec_ptr[order[k]] + l % p; e < rec_ptr[order[k] + 1]; e += p) left[l].push_back((uint32_t)e);
    }
    for (uint32_t s = 0; s < groups[w] * 4; ++s)
      for (uint32_t half = 0; half < 2; ++half) {
        uint32_t used[64] = {};
        for (uint32_t x = 0; x < 32; ++x) {
          const uint32_t l = half * 32 + (x + s) % 32;  // no lane always chooses last
          if (left[l].empty()) continue;
          const uint32_t n = (uint32_t)left[l].size(), look = std::min(n, kLook);
          uint32_t best = n - 1;
          for (uint32_t q = 0; q < look; ++q) {
            const uint32_t at = n - 1 - q;
            if (used[rec_col[left[l][at]] & 63] < used[rec_col[left[l][best]] & 63]) best = at;
            if (used[rec_col[left[l][best]] & 63] == 0) break;
          }
          const uint32_t e = left[l][best];
          left[l][best] = left[l].back();
          left[l].pop_back();
          ++used[rec_col[e] & 63];
          const size_t at = ((size_t)(s / 4) * n_thr + w * 64 + l) * 4 + s % 4;
          col[at] = (uint16_t)(rec_col[e] * 4);
          pos[e] = (uint32_t)at;
        }
      }
  }
  snn_network *pool = &pl->pool;
  a.seq_p = p;
  a.seq_max = g_max;
  a.seq_more_all = more_all;
  // one array, one copy
  std::vector<uint32_t> all(row);
  all.insert(all.end(), groups.begin(), groups.end());
  all.insert(all.end(), more.begin(), more.end());
  const size_t at_col = all.size();
  all.resize(at_col + places / 2);
  std::memcpy(all.data() + at_col, col.data(), places * sizeof(uint16_t));
  all.insert(all.end(), pos.begin(), pos.end());
  const uint32_t *dev = upload(pool, all);
  a.seq_row = dev;
  a.seq_groups = dev + n_thr;
  a.seq_more = a.seq_groups + groups.size();
  a.seq_col = reinterpret_cast<const uint16_t *>(dev + at_col);
  a.seq_pos = dev + at_col + places / 2;
  a.seq_w = dev_array<float>(pool, places);
  check(hipMemsetAsync(a.seq_w, 0, places * 4, pool->stream), "clear weights");
  check(hipStreamSynchronize(pool->stream), "sync");  // the vectors end here
  a.seq_threads = n_thr;
}

// Whether the sliced adjoint (k_adjoint_slice) is the faster one of plans without the
// event-driven form.  It is where the device holds a step's workgroups at once; further rounds
// stage the slices of all neurons again, and a wavefront per neuron (k_adjoint_step) is faster
// except with few synapses, whose gathers are short.  us per step, spiking, a wavefront per neuron
// against slices: 256 workgroups of 4,096 neurons 17.2 against 14.1 with rows of 100, 45.5 against
// 30.3 with 400; 1.1 to 1.5 rounds (2,300 neurons x 64, 3,000 x 24, 4,096 x 24) 12.9 to 14.7 against
// 11.2 to 13.4 with rows of 20, 12.3 to 14.1 against 11.8 to 14.2 with 30, 11.8 to 13.6 against
// 12.4 to 14.5 with 40 and 13.8 to 17.0 against 15.7 to 19.1 with 100; 2.9 rounds (3,000 x 64) 13.8
// against 14.7 with 20 and 14.9 against 22.3 with 100.
bool slices_fit(const snn::BpttArgs &a) {
  int device = 0, cus = 0, lds = 0;
  check(hipGetDevice(&device), "hipGetDevice");
  check(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device), "CU count");
  check(hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, device), "LDS limit");
  const uint64_t held = (uint64_t)cus * std::min<uint64_t>(2, (uint64_t)lds / (a.H * 32ull));
  const uint64_t blocks = (uint64_t)((a.B + 7) / 8) * ((a.H + snn::kAdjointRows - 1) / snn::kAdjointRows);
  return blocks <= held || (blocks <= 2 * held && a.nnz_rec <= 32ull * a.H);
}

void build_bptt(snn_bptt *p, const uint64_t *in_ptr, const int32_t *in_col, const uint64_t *rec_ptr,
                const int32_t *rec_col) {
  const snn_bptt_desc &d = p->desc;
  if (d.batch < 1 || d.batch > 64) fail(SNN_E_INVALID, "batch must be 1..64");
  if (d.steps < 1 || d.n_in < 1 || d.n_hidden < 1 || d.n_out < 1) fail(SNN_E_INVALID, "empty dimension");
  if (d.steps > 65535) fail(SNN_E_INVALID, "at most 65,535 steps");
  if (d.checkpoint < 1 || d.checkpoint > 32) fail(SNN_E_INVALID, "checkpoint interval must be 1..32");
  if (d.n_out > 1024) fail(SNN_E_INVALID, "at most 1024 readouts");
  if (!(d.slope > 0.f) || !(d.beta >= 0.f) || !(d.beta_out >= 0.f)) fail(SNN_E_INVALID, "invalid constants");
  const uint64_t nnz_in = in_ptr ? in_ptr[d.n_in] : 0, nnz_rec = rec_ptr ? rec_ptr[d.n_hidden] : 0;
  check_csr(in_ptr, in_col, d.n_in, d.n_hidden, nnz_in, "input weights");
  check_csr(rec_ptr, rec_col, d.n_hidden, d.n_hidden, nnz_rec, "recurrent weights");
  std::vector<uint64_t> it_ptr, rt_ptr;
  std::vector<int32_t> it_src, rt_src;
  std::vector<uint32_t> it_edge, rt_edge;
  transpose_csr(in_ptr, in_col, d.n_in, d.n_hidden, it_ptr, it_src, it_edge);
  transpose_csr(rec_ptr, rec_col, d.n_hidden, d.n_hidden, rt_ptr, rt_src, rt_edge);
  snn::BpttArgs &a = p->args;
  snn_network *pool = &p->pool;
  a.B = d.batch;
  a.T = d.steps;
  a.C = d.n_in;
  a.H = d.n_hidden;
  a.O = d.n_out;
  a.K = d.checkpoint;
  a.beta = d.beta;
  a.beta_out = d.beta_out;
  a.theta = d.theta;
  a.slope = d.slope;
  a.smooth = d.smooth ? 1u : 0u;
  a.detach_reset = d.smooth ? 0u : 1u;
  a.nnz_in = nnz_in;
  a.nnz_rec = nnz_rec;
  a.in_t_ptr = upload(pool, it_ptr);
  a.in_t_src = upload(pool, it_src);
  a.in_t_edge = upload(pool, it_edge);
  a.rec_t_ptr = upload(pool, rt_ptr);
  a.rec_t_src = upload(pool, rt_src);
  a.rec_t_edge = upload(pool, rt_edge);
  a.rec_ptr = upload(pool, std::vector<uint64_t>(rec_ptr, rec_ptr + d.n_hidden + 1));
  a.rec_col = upload(pool, std::vector<int32_t>(rec_col, rec_col + nnz_rec));
  const size_t HB = (size_t)a.H * 64, n_seg = (a.T + a.K - 1) / a.K;
  // 8 readable entries past the end, and for the spike masks 8 before the start: the
  // forward's input currents and the backward's segment currents read 8 steps of masks
  // per load, the latter from step t - 1 (whose values at t = 0 are not used)
  a.xbits = dev_array<uint64_t>(pool, (size_t)a.C * a.T + 8);
  a.sbits = dev_array<uint64_t>(pool, (size_t)a.H * a.T + 16) + 8;
  a.sbits_t = dev_array<uint64_t>(pool, (size_t)a.T * a.H);
  uint64_t max_deg = 0;
  for (uint32_t j = 0; j < a.H; ++j) max_deg = std::max<uint64_t>(max_deg, rt_ptr[j + 1] - rt_ptr[j]);
  snn::BpttLayouts lay{};
  a.ell_w = 0;
  a.Hp = (a.H + 255) / 256 * 256;
  a.nw = (a.H + 63) / 64;
  a.events = !a.smooth && a.H <= snn::kEventMaxNeurons && (uint64_t)a.C * a.Hp <= snn::kEventMaxInput ? 1u : 0u;
  if (a.events) {
    // dense rows of both weight matrices and the target-major pairs of W_rec
    a.col_w = (uint32_t)max_deg;
    a.in_pos = lay.in_pos = dev_array<uint32_t>(pool, nnz_in);
    a.rec_pos = lay.rec_pos = dev_array<uint32_t>(pool, nnz_rec);
    a.col_pos = lay.col_pos = dev_array<uint32_t>(pool, nnz_rec);
    const size_t n_pair = (size_t)a.col_w * a.Hp;
    a.col_pair = dev_array<uint2>(pool, n_pair);
    check(hipMemsetAsync(a.col_pair, 0, n_pair * sizeof(uint2), pool->stream), "clear padding");
    const size_t n_in = (size_t)a.C * a.Hp, n_rec = (size_t)a.H * a.Hp;
    a.dense_in = dev_array<float>(pool, n_in);
    a.dense_rec = dev_array<float>(pool, n_rec);
    check(hipMemsetAsync(a.dense_in, 0, n_in * 4, pool->stream), "clear dense weights");
    check(hipMemsetAsync(a.dense_rec, 0, n_rec * 4, pool->stream), "clear dense weights");
    a.vall = dev_array<float>(pool, (size_t)a.B * a.T * a.Hp);
    a.spk = dev_array<uint64_t>(pool, (size_t)a.B * a.T * a.nw);
    a.lists = dev_array<uint16_t>(pool, snn::bptt_lists(a) * snn::bptt_list_stride());
    a.list_len = dev_array<uint32_t>(pool, snn::bptt_lists(a));
    p->activity = a.act_out = slot_take();
  }
  // padded rows of the recurrent weights for the sliced adjoint
  uint64_t max_row = 0;
  for (uint32_t i = 0; i < a.H; ++i) max_row = std::max<uint64_t>(max_row, rec_ptr[i + 1] - rec_ptr[i]);
  const uint64_t adj_w = std::max<uint64_t>(16, (max_row + 15) / 16 * 16);
  if (a.H <= snn::kSliceMaxNeurons && adj_w * a.H <= snn::kSliceMaxPairs && (a.events || slices_fit(a))) {
    a.S = (a.B + 7) / 8;
    a.adj_w = (uint32_t)adj_w;
    const size_t n_pair = (size_t)a.H * adj_w;
    a.adj_pair = dev_array<uint2>(pool, n_pair);
    check(hipMemsetAsync(a.adj_pair, 0, n_pair * sizeof(uint2), pool->stream), "clear padding");
    a.adj_pos = lay.adj_pos = dev_array<uint32_t>(pool, nnz_rec);
    a.adj_len = lay.adj_len = dev_array<uint32_t>(pool, a.H);
  }
  build_seq(p, rec_ptr, rec_col);
  check(snn::bptt_prepare(a), "bptt prepare");
  a.flags = dev_array<uint32_t>(pool, 4);
  a.w_in_t = dev_array<float>(pool, std::max<uint64_t>(1, nnz_in));
  a.w_rec_t = dev_array<float>(pool, std::max<uint64_t>(1, nnz_rec));
  if (!a.S) a.w_rec_c = dev_array<float>(pool, std::max<uint64_t>(1, nnz_rec));
  a.w_out_c = dev_array<float>(pool, (size_t)a.H * a.O);
  a.xt = dev_array<float>(pool, (size_t)a.T * a.C * 64);
  if (!a.events) {  // the event-driven form keeps its trajectory in vall and spk
    a.iin = dev_array<float>(pool, (size_t)a.T * HB);
    a.s = dev_array<float>(pool, (size_t)a.T * HB);
    a.vtmp = dev_array<float>(pool, 2 * HB);
    a.vseg = dev_array<float>(pool, (size_t)a.K * HB);
  }
  a.vck = dev_array<float>(pool, n_seg * HB);
  a.ro = dev_array<float>(pool, (size_t)a.T * a.O * 64);
  a.lamu = dev_array<float>(pool, (size_t)a.T * a.O * 64);
  a.lamv = dev_array<float>(pool, a.S ? (size_t)a.T * a.S * a.H * 8 : (size_t)a.T * HB);
  a.lam_carry = dev_array<float>(pool, HB);
  if (a.events) a.sg = dev_array<float>(pool, (size_t)a.T * a.S * a.H * 8);
  a.m = dev_array<float>(pool, (size_t)a.B * a.O);
  a.dm = dev_array<float>(pool, (size_t)a.B * a.O);
  a.tmax = dev_array<int32_t>(pool, (size_t)a.B * a.O);
  // ELL copy of the recurrent in-edges for the hidden steps (rows padded to a multiple of
  // 64, at most 256 wide, and at most 8,192 neurons, whose masks a workgroup stages)
  if (nnz_rec && max_deg <= snn::kEllMaxWidth && a.H <= snn::kEllMaxNeurons) {
    a.ell_w = (uint32_t)((max_deg + 63) / 64 * 64);
    const size_t places = (size_t)a.H * a.ell_w;
    a.ell_src = lay.ell_src = dev_array<int32_t>(pool, places);
    a.ell_edge = lay.ell_edge = dev_array<uint32_t>(pool, places);
    a.ell_len = lay.ell_len = dev_array<uint32_t>(pool, a.H);
    a.ell_wt = dev_array<float>(pool, places);
  }
  // these layouts are made on the device from the CSR forms
  check(snn::bptt_fill_layouts(a, lay, pool->stream), "weight layouts");
  check(hipStreamSynchronize(pool->stream), "sync after plan");
}

// Runs a pass's body: from its HIP graph (captured on the first call, on the call's
// stream), or launched kernel by kernel when the plan is eager.
template <typename F>
void bptt_body(snn_bptt *p, hipGraphExec_t &exec, hipStream_t s, F &&body) {
  if (p->desc.eager) {
    check(body(s), "bptt launch");
    return;
  }
  if (!exec) {
    hipGraph_t g = nullptr;
    check(hipStreamBeginCapture(s, hipStreamCaptureModeRelaxed), "begin capture");
    const hipError_t e = body(s);
    const hipError_t e2 = hipStreamEndCapture(s, &g);
    if (e != hipSuccess || e2 != hipSuccess) {
      if (g) (void)hipGraphDestroy(g);
      check(e != hipSuccess ? e : e2, "bptt capture");
    }
    const hipError_t e3 = hipGraphInstantiate(&exec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    check(e3, "bptt graph instantiate");
  }
  check(hipGraphLaunch(exec, s), "bptt graph launch");
}

// us of a forward pass's input currents and hidden steps: the quiet form with `inputs` nonzero
// inputs and `spikes` hidden spikes per step and batch element, and the busy form.  The quiet form
// (k_input_rows, k_hidden_seq) pays for every input and spike with a row of weights, or, past
// twice the longest column, for the columns; the busy form (k_input_current, k_hidden_step_busy) for
// every synapse and launch.  64 x 250 x 700 -> 1,024 with rows of 102, at 4 / 43 / 76 / 208 / 302
// spikes: quiet 467 / 1,850 / 2,833 / 6,929 / 4,553 us, busy 1,834 / 1,859 / 1,873 / 1,944 / 1,996
// (whole forward passes); the two are equal at 43 spikes, at 33 of 201 neurons, at 42 of 500, 66 of
// 2,048, 20 of 1,024 with rows of 20 and 135 with rows of 512, where this model has 43, 28, 35, 57,
// 23 and 115.
double bptt_quiet_us(const snn::BpttArgs &a, double inputs, double spikes) {
  const bool wide = a.Hp > 1024;
  const double row = a.Hp <= 256 ? 0.10 : wide ? 0.18 : 0.14, column = wide ? 0.23 : 0.115;
  const double step = 0.6 + (spikes > 2.0 * a.col_w ? a.col_w * column : spikes * row);
  return inputs * a.B * a.T * a.Hp * 0.2e-6 + a.T * step;
}
double bptt_busy_us(const snn::BpttArgs &a, bool binary) {
  const double degree = (double)a.nnz_rec / a.H;
  return (binary ? (double)a.nnz_in * a.T * 6e-6 : 0.0) + a.T * (2.8 + 0.6e-3 * a.H + degree * (a.Hp > 1024 ? 0.034 : 0.026));
}

// Whether the next forward pass takes the busy form (event-driven plans): the faster one at the
// activity of the latest finished pass that the host has seen (0 before the first); the results
// are the same.
bool bptt_busy(const snn_bptt *p) {
  const snn::BpttArgs &a = p->args;
  if (!a.events) return false;
  // bits per word: of an input and step over the batch, of 64 neurons
  const double inputs = (double)p->activity[0] / snn::kActSamples * a.C / a.B;
  const double spikes = (double)p->activity[1] / snn::kActSamples * a.nw;
  // (inputs other than 0 and 1 take neither form's way to the input currents)
  const bool binary = p->activity[2] == 0;
  return bptt_quiet_us(a, binary ? inputs : 0.0, spikes) > bptt_busy_us(a, binary);
}

// A graph of the plan's cannot be launched into a stream that is being captured.
bool capturing(hipStream_t s) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(s, &status) != hipSuccess || status != hipStreamCaptureStatusNone;
}

void bptt_release_graphs(snn_bptt *p) {
  if (p->g_fwd) (void)hipGraphExecDestroy(p->g_fwd);
  if (p->g_bwd) (void)hipGraphExecDestroy(p->g_bwd);
  p->g_fwd = p->g_bwd = nullptr;
}

}  // namespace

extern "C" {

snn_status snn_build_network(const snn_params *prm, const snn_population *pops, uint32_t n_pops,
                             const snn_projection *proj, uint32_t n_proj, const snn_allocator *alloc,
                             void *stream, snn_network **out) {
  return guarded([&] {
    if (!prm || !out || (!pops && n_pops) || (!proj && n_proj)) fail(SNN_E_INVALID, "null argument");
    *out = nullptr;
    snn_network *net = new snn_network();
    try {
      net->prm = *prm;
      net->pops.assign(pops, pops + n_pops);
      net->proj.assign(proj, proj + n_proj);
      if (alloc && alloc->alloc && alloc->free) {
        net->alloc = *alloc;
        net->has_alloc = true;
      }
      check(hipGetDevice(&net->device), "hipGetDevice");
      hipDeviceProp_t props;
      check(hipGetDeviceProperties(&props, net->device), "hipGetDeviceProperties");
      net->cu_count = (uint32_t)std::max(1, props.multiProcessorCount);
      int lds_max = 0;
      check(hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, net->device), "LDS limit");
      net->lds_limit = (uint32_t)std::max(0, lds_max);
      if (stream) {
        net->stream = (hipStream_t)stream;
      } else {
        net->stream = stream_take(net->device);
        net->own_stream = true;
      }
      const auto t0 = std::chrono::steady_clock::now();
      build(net);
      net->build_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    } catch (...) {
      release(net);
      delete net;
      throw;
    }
    *out = net;
  });
}

snn_status snn_spacing_gaps(const uint32_t *words, uint64_t n, uint32_t *gaps, void *stream) {
  return guarded([&] {
    if (n && (!words || !gaps)) fail(SNN_E_INVALID, "null argument");
    check(snn::launch_spacing_gaps(words, n, gaps, (hipStream_t)stream), "spacing gaps launch");
  });
}

snn_status snn_step(snn_network *net) {
  return guarded([&] {
    if (!net) fail(SNN_E_INVALID, "null network");
    refuse_member(net);
    issue_window(net, 1);
  });
}

snn_status snn_run(snn_network *net, uint32_t n_steps) {
  return guarded([&] {
    if (!net) fail(SNN_E_INVALID, "null network");
    refuse_member(net);
    run(net, n_steps);
  });
}

snn_status snn_get_route(snn_network *net, uint32_t *out) {
  return guarded([&] {
    if (!net || !out) fail(SNN_E_INVALID, "null argument");
    refuse_member(net);
    *out = route(net);
  });
}

snn_status snn_memory_cache_stats(int device, uint64_t *bytes, uint64_t *blocks, uint64_t *hits,
                                  uint64_t *misses) {
  return guarded([&] {
    std::lock_guard<std::mutex> lock(g_pool_mutex);
    uint64_t b = 0, n = 0;
    for (const PoolBlock &k : g_pool)
      if (k.device == device) {
        b += k.bytes;
        ++n;
      }
    const PoolStats st = g_pool_stats.count(device) ? g_pool_stats[device] : PoolStats{};
    if (bytes) *bytes = b;
    if (blocks) *blocks = n;
    if (hits) *hits = st.hits;
    if (misses) *misses = st.misses;
  });
}

snn_status snn_memory_cache_release(int device) {
  return guarded([&] {
    pool_release(device);
    stage_release();
    slot_release();
    stream_release(device);
  });
}

snn_status snn_sync(snn_network *net) {
  return guarded([&] {
    if (!net) fail(SNN_E_INVALID, "null network");
    sync(net);
    measure_spikes(net);
  });
}

snn_status snn_get_raster_bits(snn_network *net, uint64_t t_begin, uint64_t t_end, uint64_t *words) {
  return guarded([&] {
    if (!net || (!words && t_end > t_begin)) fail(SNN_E_INVALID, "null argument");
    raster_range_check(net, t_begin, t_end);
    copy_raster_rows(net, t_begin, t_end, words);
  });
}

snn_status snn_get_raster(snn_network *net, uint64_t t_begin, uint64_t t_end, uint32_t *steps,
                          uint32_t *ids, uint64_t capacity, uint64_t *n_spikes) {
  return guarded([&] {
    if (!net || !n_spikes) fail(SNN_E_INVALID, "null argument");
    raster_range_check(net, t_begin, t_end);
    download_pairs(net, t_begin, t_end, steps, ids, capacity, n_spikes);
  });
}

snn_status snn_get_info(snn_network *net, snn_info *info) {
  return guarded([&] {
    if (!net || !info) fail(SNN_E_INVALID, "null argument");
    lazy_flush(net);  // pending potentiation counted as touches
    const CtlTotals c = read_ctl(net);
    if (c.lazy_overrun) fail(SNN_E_STATE, "lazy plasticity: a row had more pending steps than the spike history holds");
    snn_info r{};
    r.n = net->n;
    r.delay = net->delay;
    r.queue_slots = net->slots;
    r.queue_groups = snn::kQueueGroups;
    r.queue_stride = net->queue_stride;
    r.input_buffers = net->n_inbuf;
    r.window = net->window;
    r.delivery = net->delivery;
    r.tiles = net->tiles;
    r.plastic = net->plastic ? 1u : 0u;
    r.raster_steps = net->raster_cap;
    r.source_weights = net->w_src ? 1u : 0u;
    r.raster_words = net->words;
    r.table_len = net->table_len;
    r.nnz = net->nnz;
    r.t = c.t;
    r.events = c.events;
    r.spikes = c.spikes;
    r.touches = c.touches;
    r.device_bytes = net->device_bytes;
    r.build_ms = net->build_ms;
    r.gen_rows_ms = net->gen_rows_ms;
    r.gen_fill_ms = net->gen_fill_ms;
    r.index_ms = net->index_ms;
    r.tile_offset_bytes = net->tile_off ? (net->tile_off16 ? 2u : 4u) : 0u;
    r.target_bytes = net->delivery == SNN_DELIVERY_TILED ? 2u : 4u;
    r.plasticity = net->lazy ? SNN_PLASTICITY_LAZY : SNN_PLASTICITY_EAGER;
    if (c.t != net->t_host) fail(SNN_E_STATE, "device step counter disagrees with the host");
    *info = r;
    measure_spikes(net);
  });
}

snn_status snn_get_state(snn_network *net, const snn_state *st) {
  return guarded([&] {
    if (!net || !st) fail(SNN_E_INVALID, "null argument");
    lazy_flush(net);  // weights as the eager form holds them
    hipStream_t s = net->stream;
    const size_t n = net->n;
    auto d2h = [&](void *dst, const void *src, size_t bytes) {
      if (dst) check(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s), "state copy");
    };
    d2h(st->v, net->v, n * 4);
    d2h(st->ref, net->ref, n * 4);
    d2h(st->input, net->input, (size_t)net->n_inbuf * n * 4);
    d2h(st->x_pre, net->x_pre, n * 4);
    d2h(st->x_post, net->x_post, n * 4);
    d2h(st->queue, net->queue, (size_t)net->slots * net->queue_stride * 4);
    if (st->queue_len)
      check(hipMemcpy2DAsync(st->queue_len, 4, net->qlen, snn::kQlenStride * 4, 4,
                             (size_t)net->slots * snn::kQueueGroups, hipMemcpyDeviceToHost, s),
            "queue counters");
    if (st->w_f32) {
      if (!net->plastic) fail(SNN_E_INVALID, "w_f32 requested from a static network");
      d2h(st->w_f32, net->w_f32, net->nnz * 4);
    }
    sync(net);
  });
}

snn_status snn_set_state(snn_network *net, const snn_state *st) {
  return guarded([&] {
    if (!net || !st) fail(SNN_E_INVALID, "null argument");
    // lazy plasticity: pending potentiation is applied with the traces it was due under;
    // the rows' traces at age are rebuilt from the new x_pre afterwards
    lazy_flush(net);
    hipStream_t s = net->stream;
    const size_t n = net->n;
    auto h2d = [&](void *dst, const void *src, size_t bytes) {
      if (src) check(hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s), "state copy");
    };
    h2d(net->v, st->v, n * 4);
    h2d(net->ref, st->ref, n * 4);
    h2d(net->input, st->input, (size_t)net->n_inbuf * n * 4);
    h2d(net->x_pre, st->x_pre, n * 4);
    h2d(net->x_post, st->x_post, n * 4);
    h2d(net->queue, st->queue, (size_t)net->slots * net->queue_stride * 4);
    // the caller's queues need not be the raster's: launches until they have arrived
    if (st->queue || st->queue_len) net->windows_from = net->t_host + net->delay + 1;
    if (st->queue_len)
      check(hipMemcpy2DAsync(net->qlen, snn::kQlenStride * 4, st->queue_len, 4, 4,
                             (size_t)net->slots * snn::kQueueGroups, hipMemcpyHostToDevice, s),
            "queue counters");
    if (st->w_f32) {
      if (!net->plastic) fail(SNN_E_INVALID, "w_f32 given to a static network");
      h2d(net->w_f32, st->w_f32, net->nnz * 4);
    }
    lazy_flush(net);
    sync(net);
  });
}

snn_status snn_get_row(snn_network *net, uint32_t i, int32_t *col, int32_t *w_q16, float *w_f32,
                       uint64_t cap, uint64_t *len) {
  return guarded([&] {
    if (!net || !len) fail(SNN_E_INVALID, "null argument");
    if (i >= net->n) fail(SNN_E_INVALID, "neuron id out of range");
    uint64_t rp[2];
    check(hipMemcpyAsync(rp, net->row_ptr + i, 16, hipMemcpyDeviceToHost, net->stream), "row ptr");
    sync(net);
    *len = rp[1] - rp[0];
    if (*len > cap) fail(SNN_E_OVERFLOW, "row longer than cap");
    if (*len == 0) return;
    if (col) check(hipMemcpyAsync(col, net->col + rp[0], *len * 4, hipMemcpyDeviceToHost, net->stream), "row");
    if (w_q16) {
      if (net->w_src) std::fill(w_q16, w_q16 + *len, net->w_src_host[i]);
      else if (!net->w_q16) fail(SNN_E_INVALID, "network has FP32 weights");
      else check(hipMemcpyAsync(w_q16, net->w_q16 + rp[0], *len * 4, hipMemcpyDeviceToHost, net->stream), "row");
    }
    if (w_f32) {
      if (!net->w_f32) fail(SNN_E_INVALID, "network has Q16 weights");
      lazy_flush(net);
      check(hipMemcpyAsync(w_f32, net->w_f32 + rp[0], *len * 4, hipMemcpyDeviceToHost, net->stream), "row");
    }
    sync(net);
  });
}

snn_status snn_get_synapses(snn_network *net, uint64_t *row_ptr, int32_t *col, int32_t *w_q16,
                            float *w_f32) {
  return guarded([&] {
    if (!net) fail(SNN_E_INVALID, "null network");
    hipStream_t s = net->stream;
    if (row_ptr) check(hipMemcpyAsync(row_ptr, net->row_ptr, ((size_t)net->n + 1) * 8, hipMemcpyDeviceToHost, s), "copy");
    if (col) check(hipMemcpyAsync(col, net->col, net->nnz * 4, hipMemcpyDeviceToHost, s), "copy");
    if (w_q16) {
      if (net->w_src) {
        std::vector<uint64_t> rp((size_t)net->n + 1);
        check(hipMemcpyAsync(rp.data(), net->row_ptr, rp.size() * 8, hipMemcpyDeviceToHost, s), "copy");
        sync(net);
        for (uint32_t i = 0; i < net->n; ++i) std::fill(w_q16 + rp[i], w_q16 + rp[i + 1], net->w_src_host[i]);
      } else if (!net->w_q16) {
        fail(SNN_E_INVALID, "network has FP32 weights");
      } else {
        check(hipMemcpyAsync(w_q16, net->w_q16, net->nnz * 4, hipMemcpyDeviceToHost, s), "copy");
      }
    }
    if (w_f32) {
      if (!net->w_f32) fail(SNN_E_INVALID, "network has Q16 weights");
      lazy_flush(net);
      check(hipMemcpyAsync(w_f32, net->w_f32, net->nnz * 4, hipMemcpyDeviceToHost, s), "copy");
    }
    sync(net);
  });
}

snn_status snn_get_drive_table(snn_network *net, uint64_t *table, uint32_t cap) {
  return guarded([&] {
    if (!net || !table) fail(SNN_E_INVALID, "null argument");
    if (cap < net->table_len) fail(SNN_E_OVERFLOW, "table longer than cap");
    std::memcpy(table, net->table, net->table_len * 8);
  });
}

snn_status snn_set_profiling(snn_network *net, int32_t on) {
  return guarded([&] {
    if (!net) fail(SNN_E_INVALID, "null network");
    net->profiling = on != 0;
  });
}

snn_status snn_get_profile(snn_network *net, snn_profile *prof) {
  return guarded([&] {
    if (!net || !prof) fail(SNN_E_INVALID, "null argument");
    resolve_profile(net);
    *prof = net->prof;
  });
}

snn_status snn_reset_profile(snn_network *net) {
  return guarded([&] {
    if (!net) fail(SNN_E_INVALID, "null network");
    resolve_profile(net);
    net->prof = snn_profile{};
  });
}

snn_status snn_time_delivery(snn_network *net, const uint32_t *ids_host, uint32_t n_ids,
                             const uint32_t *step_counts, uint32_t steps, uint32_t reps,
                             double *avg_ms, uint64_t *events) {
  return guarded([&] {
    if (!net || (!ids_host && n_ids) || !avg_ms) fail(SNN_E_INVALID, "null argument");
    refuse_member(net);
    if (steps == 0) steps = net->window;
    if (steps > net->window) fail(SNN_E_INVALID, "steps exceeds the network's window");
    std::vector<std::vector<uint32_t>> per_step(steps);
    if (step_counts) {
      uint64_t k = 0;
      for (uint32_t w = 0; w < steps; ++w) {
        if (k + step_counts[w] > n_ids) fail(SNN_E_INVALID, "step counts exceed the ids");
        per_step[w].assign(ids_host + k, ids_host + k + step_counts[w]);
        k += step_counts[w];
      }
      if (k != n_ids) fail(SNN_E_INVALID, "step counts do not sum to n_ids");
    } else {
      for (uint32_t k = 0; k < n_ids; ++k) per_step[k % steps].push_back(ids_host[k]);
    }
    uint64_t ev = 0;
    *avg_ms = time_delivery(net, per_step, reps, &ev);
    if (events) *events = ev;
  });
}

snn_status snn_time_delivery_static(snn_network *net, const uint32_t *ids_host, uint32_t n_ids,
                                    const uint32_t *step_counts, uint32_t steps, uint32_t reps,
                                    double *avg_ms, uint64_t *events) {
  return guarded([&] {
    if (!net || (!ids_host && n_ids) || !avg_ms) fail(SNN_E_INVALID, "null argument");
    refuse_member(net);
    if (steps == 0) steps = net->window;
    *avg_ms = time_delivery_static(net, ids_host, n_ids, step_counts, steps, reps, events);
  });
}

snn_status snn_set_delivery(snn_network *net, uint32_t delivery, uint32_t tiles, uint32_t block, uint32_t grid) {
  return guarded([&] {
    if (!net) fail(SNN_E_INVALID, "null network");
    refuse_member(net);
    set_delivery(net, delivery, tiles, block, grid, true);
  });
}

snn_status snn_autotune_delivery(snn_network *net, uint32_t reps, snn_delivery_tuning *chosen) {
  return guarded([&] {
    if (!net) fail(SNN_E_INVALID, "null network");
    refuse_member(net);
    const snn_delivery_tuning t = autotune_delivery(net, reps);
    if (chosen) *chosen = t;
  });
}

void snn_destroy(snn_network *net) {
  if (!net || net->owner) return;
  try {
    resolve_profile(net);
  } catch (...) {
  }
  release(net);
  delete net;
}

const char *snn_last_error(const snn_network *) { return g_error.c_str(); }

snn_status snn_build_batch(const snn_batch_member *nets, uint32_t n_nets, uint32_t raster_steps,
                           const snn_allocator *alloc, void *stream, snn_batch **out) {
  return guarded([&] {
    if (!out || (!nets && n_nets)) fail(SNN_E_INVALID, "null argument");
    *out = nullptr;
    if (n_nets == 0) fail(SNN_E_INVALID, "a batch needs at least one network");
    snn_batch *b = new snn_batch();
    try {
      if (alloc && alloc->alloc && alloc->free) {
        b->pool.alloc = *alloc;
        b->pool.has_alloc = true;
      }
      check(hipGetDevice(&b->pool.device), "hipGetDevice");
      hipDeviceProp_t props;
      check(hipGetDeviceProperties(&props, b->pool.device), "hipGetDeviceProperties");
      b->pool.cu_count = (uint32_t)std::max(1, props.multiProcessorCount);
      if (stream) {
        b->pool.stream = (hipStream_t)stream;
      } else {
        b->pool.stream = stream_take(b->pool.device);
        b->pool.own_stream = true;
      }
      build_batch(b, nets, n_nets, raster_steps);
    } catch (...) {
      batch_destroy(b);
      delete b;
      throw;
    }
    *out = b;
  });
}

snn_status snn_batch_run(snn_batch *b, uint32_t n_steps) {
  return guarded([&] {
    if (!b) fail(SNN_E_INVALID, "null batch");
    batch_run(b, n_steps);
  });
}

snn_status snn_batch_sync(snn_batch *b) {
  return guarded([&] {
    if (!b) fail(SNN_E_INVALID, "null batch");
    check(hipStreamSynchronize(b->pool.stream), "stream sync");
  });
}

snn_status snn_batch_network(snn_batch *b, uint32_t k, snn_network **net) {
  return guarded([&] {
    if (!b || !net) fail(SNN_E_INVALID, "null argument");
    if (k >= b->nets.size()) fail(SNN_E_INVALID, "member index out of range");
    *net = b->nets[k];
  });
}

snn_status snn_batch_autotune(snn_batch *b, uint32_t trial_steps, snn_batch_tuning *chosen) {
  return guarded([&] {
    if (!b) fail(SNN_E_INVALID, "null batch");
    const snn_batch_tuning t = batch_autotune(b, trial_steps);
    if (chosen) *chosen = t;
  });
}

snn_status snn_batch_set_tuning(snn_batch *b, const snn_batch_tuning *tuning) {
  return guarded([&] {
    if (!b || !tuning) fail(SNN_E_INVALID, "null argument");
    check(hipStreamSynchronize(b->pool.stream), "stream sync");
    batch_apply_tuning(b, *tuning);
  });
}

snn_status snn_batch_get_tuning(snn_batch *b, snn_batch_tuning *tuning) {
  return guarded([&] {
    if (!b || !tuning) fail(SNN_E_INVALID, "null argument");
    *tuning = b->tuning;
  });
}

void snn_batch_destroy(snn_batch *b) {
  if (!b) return;
  batch_destroy(b);
  delete b;
}

snn_status snn_bptt_create(const snn_bptt_desc *desc, const uint64_t *in_row_ptr, const int32_t *in_col,
                           const uint64_t *rec_row_ptr, const int32_t *rec_col, const snn_allocator *alloc,
                           void *stream, snn_bptt **out) {
  return guarded([&] {
    if (!desc || !out || !in_row_ptr || !rec_row_ptr) fail(SNN_E_INVALID, "null argument");
    *out = nullptr;
    snn_bptt *p = new snn_bptt();
    try {
      p->desc = *desc;
      if (alloc && alloc->alloc && alloc->free) {
        p->pool.alloc = *alloc;
        p->pool.has_alloc = true;
      }
      check(hipGetDevice(&p->pool.device), "hipGetDevice");
      if (stream) {
        p->pool.stream = (hipStream_t)stream;
      } else {
        p->pool.stream = stream_take(p->pool.device);
        p->pool.own_stream = true;
      }
      build_bptt(p, in_row_ptr, in_col, rec_row_ptr, rec_col);
    } catch (...) {
      release(&p->pool);
      delete p;
      throw;
    }
    *out = p;
  });
}

snn_status snn_bptt_forward(snn_bptt *p, const float *x, const float *w_in, const float *w_rec,
                            const float *w_out, const int32_t *labels, float *loss, void *stream) {
  return guarded([&] {
    if (!p || !x || !w_out || !labels || !loss || (!w_in && p->args.nnz_in) || (!w_rec && p->args.nnz_rec))
      fail(SNN_E_INVALID, "null argument");
    snn::BpttArgs a = p->args;
    a.w_in = w_in;
    a.w_rec = w_rec;
    a.w_out = w_out;
    hipStream_t s = stream ? (hipStream_t)stream : p->pool.stream;
    const bool busy = bptt_busy(p) && (p->desc.eager || !capturing(s));
    check(snn::bptt_forward_prologue(a, x, busy, s), "bptt forward");
    snn::BpttArgs g = p->args;  // the body reads the plan's buffers only
    g.w_out = g.w_out_c;
    if (a.events && !busy) check(snn::bptt_hidden_seq(a, s), "bptt forward");
    else bptt_body(p, p->g_fwd, s, [&](hipStream_t st) { return snn::bptt_forward_body(g, st); });
    if (a.events) check(snn::bptt_readout_events(a, busy, s), "bptt forward");
    check(snn::bptt_forward_epilogue(a, labels, loss, s), "bptt forward");
    p->forwards++;
  });
}

snn_status snn_bptt_get_route(snn_bptt *p, uint32_t *out) {
  return guarded([&] {
    if (!p || !out) fail(SNN_E_INVALID, "null argument");
    *out = p->args.events && !bptt_busy(p) ? SNN_ROUTE_PERSISTENT : SNN_ROUTE_LAUNCHES;
  });
}

snn_status snn_bptt_backward(snn_bptt *p, const float *w_in, const float *w_rec, const float *w_out,
                             const float *g_loss, float *g_w_in, float *g_w_rec, float *g_w_out,
                             void *stream) {
  return guarded([&] {
    if (!p || !w_out || !g_w_out || (!w_in && p->args.nnz_in) || (!w_rec && p->args.nnz_rec) ||
        (!g_w_in && p->args.nnz_in) || (!g_w_rec && p->args.nnz_rec))
      fail(SNN_E_INVALID, "null argument");
    if (p->forwards == 0) fail(SNN_E_STATE, "backward before any forward pass");
    snn::BpttArgs a = p->args;
    a.w_in = w_in;
    a.w_rec = w_rec;
    a.w_out = w_out;
    a.g_w_in = g_w_in;
    a.g_w_rec = g_w_rec;
    a.g_w_out = g_w_out;
    hipStream_t s = stream ? (hipStream_t)stream : p->pool.stream;
    check(snn::bptt_backward_prologue(a, g_loss, s), "bptt backward");
    if (a.seq_threads) {  // a few kernels, on the caller's weights
      check(snn::bptt_backward_body(a, s), "bptt backward");
      check(snn::bptt_backward_epilogue(a, s), "bptt backward");
      return;
    }
    snn::BpttArgs g = p->args;
    g.w_out = g.w_out_c;
    g.w_rec = g.w_rec_c;
    bptt_body(p, p->g_bwd, s, [&](hipStream_t st) { return snn::bptt_backward_body(g, st); });
    check(snn::bptt_backward_epilogue(a, s), "bptt backward");
  });
}

snn_status snn_bptt_get_trace(snn_bptt *p, float *spikes, float *v_checkpoints, float *readout_max,
                              int32_t *readout_argmax, void *stream) {
  return guarded([&] {
    if (!p) fail(SNN_E_INVALID, "null plan");
    const snn::BpttArgs &a = p->args;
    hipStream_t s = stream ? (hipStream_t)stream : p->pool.stream;
    const size_t HB = (size_t)a.H * 64, n_seg = (a.T + a.K - 1) / a.K;
    std::vector<uint64_t> masks;
    if (a.events) {
      if (v_checkpoints) check(snn::bptt_trace_v(a, s), "trace");
      if (spikes) {
        check(snn::bptt_spike_masks(a, s), "trace");
        masks.resize((size_t)a.H * a.T);
        check(hipMemcpyAsync(masks.data(), a.sbits, masks.size() * 8, hipMemcpyDeviceToHost, s), "copy");
      }
    } else if (spikes) {
      check(hipMemcpyAsync(spikes, a.s, (size_t)a.T * HB * 4, hipMemcpyDeviceToHost, s), "copy");
    }
    if (v_checkpoints) check(hipMemcpyAsync(v_checkpoints, a.vck, n_seg * HB * 4, hipMemcpyDeviceToHost, s), "copy");
    if (readout_max) check(hipMemcpyAsync(readout_max, a.m, (size_t)a.B * a.O * 4, hipMemcpyDeviceToHost, s), "copy");
    if (readout_argmax)
      check(hipMemcpyAsync(readout_argmax, a.tmax, (size_t)a.B * a.O * 4, hipMemcpyDeviceToHost, s), "copy");
    check(hipStreamSynchronize(s), "sync");
    if (!masks.empty())  // the event-driven form holds spikes as batch masks
      for (uint32_t t = 0; t < a.T; ++t)
        for (uint32_t i = 0; i < a.H; ++i)
          for (uint32_t b = 0; b < 64; ++b)
            spikes[((size_t)t * a.H + i) * 64 + b] = (float)((masks[(size_t)i * a.T + t] >> b) & 1u);
  });
}

void snn_bptt_destroy(snn_bptt *p) {
  if (!p) return;
  if (p->pool.stream) (void)hipStreamSynchronize(p->pool.stream);
  bptt_release_graphs(p);
  release(&p->pool);
  delete p;
}

}  // extern "C"
