// plastic.hip -- windows of steps of an eagerly plastic network.
//
// Within `delay` steps nothing that a target does reaches another target: the spikes that
// arrive in the steps [t0, t0 + d) were emitted before t0, and a synapse i -> j changes with
// i's arrivals (known at t0), with j's own spikes and with j's own trace.  So a workgroup
// that owns a range of targets runs a whole window of up to d - 1 steps by itself, with
// workgroup barriers between the phases and no other synchronisation.  Depression of step
// t + 1 needs the trace of step t only, so it is applied where the row is delivered;
// potentiation waits until the row arrives again or the window ends.  Every synapse sees the
// same binary32 operations in the same order as in the launch-per-phase form (update,
// plasticity, delivery), so weights, traces, input and counters are the same bit for bit.
//
// Two launches per window:
//  k_plastic_prepare  potentiation left by the window before; per neuron the presynaptic
//                     trace at t0 and a mask of the arrivals in the window (a synapse's
//                     trace at any step follows from there); and the targets of the rows that
//                     arrive, read whole and laid out per range.
//  k_plastic_window   the steps.
//
// Bound: scattered lines of memory.  A compute unit keeps about 64 line reads in flight, so
// what counts is the number of lines and that all units have the same number to read: 1.4
// lines per sub-row (weights, a part of a line of targets) in the window launch, two per
// potentiated synapse (weight, its source's trace) in the prepare launch.  A window of nine
// steps of 100,000 neurons (2e8 synapses) takes 34 + 61 us in a trace of 8,300 steps, start-up
// burst included, one of 10,000 neurons (45 spikes a step) 17 + 9 us; by the clock 14 us a step
// at 120 spikes a step and 2.9, where update, plasticity and delivery launches take 30 and 16.
//
// k_plastic_import and k_plastic_export take the spikes to and from the FIFO ring's form at
// both ends of a run.
#include <algorithm>

#include "device_math.h"
#include "snn_internal.h"

namespace snn {
namespace {

constexpr int kPrepBlock = 256;
constexpr int kPrepWaves = kPrepBlock / kWave;
constexpr uint32_t kPrepRanges = 512;
constexpr uint32_t kPlasticTarget = 0x8000u;  // flag of a laid-out target: its synapse is plastic
constexpr int kListBlock = 1024;
constexpr int kT = kPlasticBlock;
constexpr int kWaves = kT / kWave;
constexpr int kU = kPlasticAhead;  // synapses of a lane in flight: delivery
constexpr int kLtp = 8;         //   potentiation
constexpr uint32_t kLtpParts = 32;
constexpr uint32_t kXcds = 8;

__device__ __forceinline__ const uint64_t *raster_row(uint64_t s, const PlasticArgs &a) {
  return a.raster + (s % a.raster_cap) * a.words;
}
__device__ __forceinline__ uint32_t *list_count(uint64_t s, const PlasticArgs &a) {
  return a.list_len + (s % a.list_slots) * kQlenStride;
}
__device__ __forceinline__ int32_t *list_ids(uint64_t s, const PlasticArgs &a) {
  return a.list + (s % a.list_slots) * a.n;
}
// Number of spikes that arrive as list m of a window from t0 on: those of step t0 - d + m.
// List 0 serves the depression of step t0; it is empty if the window before has done that.
__device__ __forceinline__ uint32_t list_length(const PlasticArgs &a, uint64_t t0, uint32_t m, uint32_t steps) {
  if (m > steps || t0 + m < a.delay || (m == 0 && !a.first)) return 0;
  return *list_count(t0 + m - a.delay, a);
}

__device__ __forceinline__ uint32_t range_bound(const PlasticArgs &a, int32_t src, uint32_t r) {
  const size_t at = (size_t)src * (a.ranges + 1) + r;
  return a.off16 ? static_cast<const uint16_t *>(a.off)[at] : static_cast<const uint32_t *>(a.off)[at];
}

__device__ __forceinline__ SubRow sub_row(const PlasticArgs &a, int32_t src, uint32_t r, uint2 trace) {
  const uint32_t o0 = range_bound(a, src, r), o1 = range_bound(a, src, r + 1);
  const uint32_t q0 = a.plast_rel[src], q1 = q0 + a.plast_len[src];
  SubRow h;
  h.lo = (uint32_t)a.row_ptr[src] + o0;
  h.dims = (o1 - o0) | (min(max(q0, o0), o1) - o0) << 10 | (min(max(q1, o0), o1) - o0) << 20;
  h.trace = trace;
  return h;
}

// Potentiation of one synapse by the spikes `pend` of its target (bit q: step t0 + q), oldest
// first; tr is its source's trace.
__device__ __forceinline__ float potentiate(const PlasticArgs &a, uint2 tr, uint32_t pend, float w) {
  float x = __uint_as_float(tr.x);
  for (uint32_t q = 0; pend >> q; ++q) {
    x = x * a.beta_plus;
    if ((tr.y >> q) & 1u) x = x + 1.0f;
    if ((pend >> q) & 1u) {
      const float dw = a.a_plus * x;
      w = w + dw;
      if (w > a.w_max) w = a.w_max;
    }
  }
  return w;
}

// A barrier that waits for LDS accesses only: loads and stores of global memory stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The potentiation that the window before has left: the in-edges of its spiking neurons, one
// writer per synapse.  Bound: a scattered read and write of a line per synapse; a compute
// unit keeps about 64 such reads in flight, so the work has to be spread over all of them
// (by the ranges' own workgroups, whose spikes vary, it took 2.5 times as long).
__device__ void left_potentiation(const PlasticArgs &a, uint32_t block, uint32_t blocks) {
  const uint32_t cnt = *a.ltp_len[a.parity ^ 1u];
  const uint32_t n_waves = blocks * kPrepWaves, lane = lane_id();
  const uint32_t parts = cnt ? min(max(n_waves / cnt, 1u), kLtpParts) : 1u;
  const uint2 *trace = a.trace[a.parity ^ 1u];
  for (uint64_t item = block * kPrepWaves + threadIdx.x / kWave; item < (uint64_t)cnt * parts; item += n_waves) {
    const uint4 spk = a.ltp[a.parity ^ 1u][item / parts];  // first in-edge, number, spikes
    const uint32_t chunk = (spk.y + parts - 1) / parts;
    const uint32_t k0 = (uint32_t)(item % parts) * chunk, k1 = min(k0 + chunk, spk.y);
    for (uint32_t kb = k0 + lane; kb < k1; kb += kLtp * kWave) {
      uint32_t edge[kLtp], src[kLtp];
      float w[kLtp];
      uint2 tr[kLtp];
#pragma unroll
      for (int u = 0; u < kLtp; ++u) {
        const uint32_t k = kb + u * kWave;
        edge[u] = src[u] = 0;
        if (k < k1) {
          edge[u] = a.in_edge[(size_t)spk.x + k];
          src[u] = (uint32_t)a.in_src[(size_t)spk.x + k];
        }
      }
#pragma unroll
      for (int u = 0; u < kLtp; ++u) {
        w[u] = 0.f;
        tr[u] = make_uint2(0, 0);
        if (kb + u * kWave < k1) {
          w[u] = a.w_f32[edge[u]];
          tr[u] = trace[src[u]];
        }
      }
#pragma unroll
      for (int u = 0; u < kLtp; ++u) {
        if (kb + u * kWave >= k1) continue;
        // what came before the source's last arrival was applied with that
        uint32_t pend = spk.z;
        if (tr[u].y) pend &= ~0u << (31u - (uint32_t)__builtin_clz(tr[u].y));
        if (pend) a.w_f32[edge[u]] = potentiate(a, tr[u], pend, w[u]);
      }
    }
  }
}

// Rows are laid out by workgroups that read them whole: a range reading its own piece of the
// targets would fetch 1.25 lines for 32 bytes at a random place, and here four sub-rows share
// a line.
//
// Workgroups: a.ltp_blocks for the potentiation left, a.row_blocks for the arriving rows, the
// others one neuron per thread.  steps == 0: potentiation only.
__global__ __launch_bounds__(kPrepBlock) void k_plastic_prepare(PlasticArgs a, uint32_t steps) {
  const uint32_t lane = lane_id();
  if (blockIdx.x < a.ltp_blocks) {
    left_potentiation(a, blockIdx.x, a.ltp_blocks);
    return;
  }
  const uint64_t t0 = a.ctl->t;
  const uint32_t block = blockIdx.x - a.ltp_blocks;
  if (block >= a.row_blocks) {
    const uint32_t i = (block - a.row_blocks) * kPrepBlock + threadIdx.x;
    if (i == 0) {
      a.ctl->t_deliver = t0;
      *a.ltp_len[a.parity] = 0;
    }
    if (i <= kPlasticSteps) a.arriving[i] = list_length(a, t0, i, steps);
    if (i < steps) *list_count(t0 + i, a) = 0;  // the window's own spikes
    if (i >= a.n) return;
    uint32_t arrivals = 0;
#pragma unroll
    for (uint32_t m = 0; m <= kPlasticSteps; ++m) {
      const uint64_t s = t0 + m;
      if (m <= steps && s >= a.delay)
        arrivals |= (uint32_t)((raster_row(s - a.delay, a)[i / kWave] >> (i % kWave)) & 1u) << m;
    }
    a.trace[a.parity][i] = make_uint2(__float_as_uint(a.x_pre[i]), arrivals);
    return;
  }
  __shared__ uint32_t s_off[kPrepRanges];  // range boundaries of a row
  // every wavefront finds the lists' lengths by itself
  const uint32_t len = list_length(a, t0, lane, steps);
  const uint32_t end = wave_inclusive_scan(len);
  const uint32_t total = min((uint32_t)__builtin_amdgcn_readlane((int)end, kWave - 1), a.row_cap);
  for (uint32_t x = block; x < total; x += a.row_blocks) {
    const uint32_t m = (uint32_t)__popcll(__ballot(end <= x));  // the list of row x
    const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)(end - len), (int)m);
    const int32_t src = list_ids(t0 + m - a.delay, a)[x - first];
    bool arrives = false;
    if (lane <= steps && t0 + lane >= a.delay)
      arrives = (raster_row(t0 + lane - a.delay, a)[(uint32_t)src / kWave] >> ((uint32_t)src % kWave)) & 1u;
    const uint2 trace = make_uint2(__float_as_uint(a.x_pre[src]), (uint32_t)__ballot(arrives));
    const uint64_t lo = a.row_ptr[src];
    const uint32_t n_syn = (uint32_t)(a.row_ptr[src + 1] - lo), q0 = a.plast_rel[src], q_len = a.plast_len[src];
    const bool held = a.ranges <= kPrepRanges;
    __syncthreads();
    if (held)
      for (uint32_t r = threadIdx.x; r < a.ranges; r += kPrepBlock) s_off[r] = range_bound(a, src, r);
    __syncthreads();
#pragma unroll 4
    for (uint32_t k = threadIdx.x; k < n_syn; k += kPrepBlock) {
      const uint32_t j = (uint32_t)a.col[lo + k];
      const uint32_t r = j / a.range;
      const uint32_t at = k - (held ? s_off[r] : range_bound(a, src, r));
      if (at >> a.lanes_shift) continue;
      a.row_tgt[(((size_t)r * a.row_cap + x) << a.lanes_shift) + at] =
          (uint16_t)((j - r * a.range) | (k - q0 < q_len ? kPlasticTarget : 0u));
    }
    for (uint32_t r = threadIdx.x; r < a.ranges; r += kPrepBlock)
      a.row_head[(size_t)r * a.row_cap + x] = sub_row(a, src, r, trace);
  }
}

struct Fetched {  // a lane's synapses of the next list, in flight
  uint32_t len[kU];   // of their sub-rows (kDirect: not fetched)
  uint32_t from[kU];  // first step whose potentiation may be pending
  uint32_t e[kU];
  uint32_t x[kU];     // target in the range
  float w[kU];
};
constexpr uint32_t kDirect = kPlasticBlock + 1;

// A workgroup per range of a.range targets, a lane per target for the update and lane groups
// per sub-row for the delivery.  The drive counts of the whole window are drawn first, by all
// wavefronts and beside the first round trips, and the next list's weights are in flight during
// the update (with the drive in the step and the lists' headers a round trip later, a window of
// 10,000 neurons took 26 instead of 18 us).  Synapses
// with potentiation pending take it here, from the trace in the row's header: going back to
// memory for it took 24 instead of 18 us per window of 10,000 neurons.
__global__ __launch_bounds__(kT) void k_plastic_window(PlasticArgs a, uint32_t steps) {
  __shared__ SubRow hdr[kPlasticRows];
  __shared__ __align__(16) uint32_t tbl[kTableCap];
  __shared__ __align__(16) uint16_t guide[kGuideBuckets];
  __shared__ uint8_t s_drive[kPlasticSteps + 6][kT];  // drive counts of the window's quads of steps
  __shared__ int32_t acc[kT];
  __shared__ float xq_next[kT];
  __shared__ uint32_t s_spk[kT];       // bit q: spike of step t0 + q
  __shared__ uint32_t s_pre[kPlasticSteps + 2];
  __shared__ uint32_t s_base[kWaves][kPlasticSteps + 1];  // places of a wavefront's spikes in the lists
  __shared__ uint32_t s_again;
  static_assert(kTableCap / 4 <= kT && kGuideBuckets / 8 == kT, "one 16-byte load of each table per lane");

  const uint64_t t0 = a.ctl->t_deliver;
  const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  // neighbouring ranges on one XCD: they share cache lines of the rows
  const uint32_t per = (a.ranges + kXcds - 1) / kXcds;
  const uint32_t r = (blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
  if (blockIdx.x / kXcds >= per || r >= a.ranges) return;
  const uint32_t lo = r * a.range;
  const uint32_t i = lo + tid;
  const bool owner = tid < a.range;  // whole wavefronts
  const bool active = owner && i < a.n;
  const bool drive = a.table_len > 1;
  const LifConst lif{a.alpha, a.v_inf, a.v_th, a.v_reset, a.ref_steps, a.w_ext_q16};

  // ---- one round trip: lengths of the lists, tables, state ----
  const uint32_t len = wave == 0 && lane <= kPlasticSteps ? a.arriving[lane] : 0u;
  const SubRow *rows_in = a.row_head + (size_t)r * a.row_cap;
  SubRow first_row{};  // of rows that may not be there
  if (tid < a.row_cap) first_row = rows_in[tid];
  if (drive) {
    if (tid < kTableCap / 4) reinterpret_cast<int4 *>(tbl)[tid] = reinterpret_cast<const int4 *>(a.table32)[tid];
    reinterpret_cast<int4 *>(guide)[tid] = reinterpret_cast<const int4 *>(a.guide)[tid];
  }
  float v = 0.f, xp = 0.f, xq = 0.f;
  int32_t ref = 0, x0 = 0;
  uint32_t arrivals = 0, in_lo = 0, in_len = 0, spikes = 0;
  if (active) {
    const uint2 tr = a.trace[a.parity][i];
    v = a.v[i];
    ref = a.ref[i];
    x0 = a.input[i];
    xq = a.x_post[i];
    xp = __uint_as_float(tr.x);
    arrivals = tr.y;
    in_lo = (uint32_t)a.in_ptr[i];
    in_len = (uint32_t)a.in_ptr[i + 1] - in_lo;
  }
  acc[tid] = x0;
  xq_next[tid] = xq * a.beta_minus;
  s_spk[tid] = 0;
  if (wave == 0) {
    const uint32_t incl = wave_inclusive_scan(len);
    if (lane <= steps) s_pre[lane + 1] = incl;
    if (lane == 0) s_pre[0] = 0;
  }
  if (tid == 0) s_again = 0;
  __syncthreads();
  uint64_t events = 0, touched = 0;
  if (drive) {
    // one Philox block per neuron and quad of steps, its word t mod 4 feeding step t
    const uint32_t quads = (((uint32_t)t0 & 3u) + steps + 3) >> 2;
    for (uint32_t x = tid; x < quads * a.range; x += kT) {
      const uint32_t q = x / a.range, c = x - q * a.range;
      const uint64_t at = (t0 >> 2) + q;
      const Words4 rnd = philox(lo + c, (uint32_t)at, (uint32_t)(at >> 32), kStreamPoisson, a.key0, a.key1);
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) {
        const uint32_t gk = guide[rnd.w[u] >> (32 - kGuideBits)];
        uint32_t k = gk & 0xFFu;
        const uint32_t k_hi = gk >> 8;
        while (k < k_hi && tbl[k] <= rnd.w[u]) ++k;
        s_drive[4 * q + u][c] = (uint8_t)k;
      }
    }
  }
  {
    const uint32_t all = s_pre[steps + 1], total = min(all, a.row_cap);
    bool again = all > a.row_cap;  // not known of the sub-rows that are not laid out
    const uint32_t ltd_end = a.last ? s_pre[steps] : all;
    auto hold = [&](uint32_t x, const SubRow &h) {
      hdr[x] = h;
      again |= h.again();
      if (x >= s_pre[1]) events += h.len();
      if (x < ltd_end) touched += h.p1() - h.p0();
    };
    if (tid < total) hold(tid, first_row);
    for (uint32_t x = tid + kT; x < total; x += kT) hold(x, rows_in[x]);
    if (again) s_again = 1;
  }
  __syncthreads();
  const bool any_again = s_again != 0;
  const uint16_t *tgt_in = a.row_tgt + (((size_t)r * a.row_cap) << a.lanes_shift);

  // Lane groups of 2^lanes_shift take a sub-row each, kU of them in flight.
  const uint32_t sub = tid & ((1u << a.lanes_shift) - 1u);
  const uint32_t lanes = 1u << a.lanes_shift, rows = kT >> a.lanes_shift;
  const uint32_t f_first = tid >> a.lanes_shift;
  auto header = [&](uint32_t m, uint32_t f) {
    const uint32_t x = s_pre[m] + f;
    if (x < a.row_cap) return hdr[x];
    const int32_t src = list_ids(t0 + m - a.delay, a)[f];
    return sub_row(a, src, r, a.trace[a.parity][src]);
  };
  // Sub-row f of list m from its memory, in general: pending potentiation, delivery (the
  // window's first step was delivered before), depression (the step after the run's last
  // window is not reached); this lane's synapses from k0 on.
  auto general = [&](uint32_t m, uint32_t f, uint32_t k0) {
    const SubRow h = header(m, f);
    const bool deliver = m > 0, ltd = m < steps || !a.last;
    for (uint32_t k = k0; k < h.len(); k += lanes) {
      const uint32_t x = (uint32_t)a.col[h.lo + k] - lo;
      const bool plastic = k >= h.p0() && k < h.p1();
      const float w = a.w_f32[h.lo + k];
      float nw = w;
      if (plastic) {
        const uint32_t pend = s_spk[x] & (~0u << h.from(m));
        if (pend) nw = potentiate(a, h.trace, pend, nw);
      }
      if (deliver) atomicAdd(&acc[x], __float2int_rn(nw * 65536.0f));
      if (plastic && ltd) {
        const float dw = a.a_minus * xq_next[x];
        nw = nw - dw;
        if (nw < 0.0f) nw = 0.0f;
      }
      if (__float_as_uint(nw) != __float_as_uint(w)) a.w_f32[h.lo + k] = nw;
    }
    if (sub == 0 && s_pre[m] + f >= a.row_cap) {  // the others were counted at the start
      if (deliver) events += h.len();
      if (ltd) touched += h.p1() - h.p0();
    }
  };
  // The weights of a row that arrives once in the window are not written before its step, so
  // its loads may run ahead; the others, and those that are not laid out, are read at their
  // step.
  Fetched ahead;
  auto fetch = [&](uint32_t m) {
    const uint32_t first = s_pre[m], cnt = s_pre[m + 1] - first;
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint32_t f = f_first + u * rows;
      ahead.len[u] = 0;
      if (u * rows < cnt && f < cnt) {  // (the first half is uniform)
        ahead.len[u] = kDirect;
        if (first + f < a.row_cap) {
          const SubRow h = hdr[first + f];
          if (!h.again()) {
            ahead.len[u] = h.len();
            ahead.from[u] = h.from(m);
            ahead.e[u] = h.lo + sub;
            if (sub < h.len()) {
              ahead.x[u] = tgt_in[((size_t)(first + f) << a.lanes_shift) + sub];
              ahead.w[u] = a.w_f32[ahead.e[u]];
            }
          }
        }
      }
    }
  };

  fetch(1);
  // depression of the first step's arrivals (the later steps' goes with their delivery)
  for (uint32_t f = f_first; f < s_pre[1]; f += rows) general(0, f, sub);
  if (any_again) __syncthreads();
  else lds_barrier();

  uint64_t my_mask = 0;  // lane w: the wavefront's spikes of step t0 + w
  uint32_t ring = (uint32_t)(t0 % a.raster_cap);
  for (uint32_t w = 0; w < steps; ++w) {
    // ---- update ----
    if (owner) {
      const int32_t x = acc[tid];
      acc[tid] = 0;
      const int32_t k = drive ? (int32_t)s_drive[((uint32_t)t0 & 3u) + w][tid] : 0;
      const bool spike = lif_advance(v, ref, x, k, lif) && active;
      xp = xp * a.beta_plus;
      if ((arrivals >> w) & 1u) xp = xp + 1.0f;
      xq = xq * a.beta_minus;
      if (spike) {
        xq = xq + 1.0f;
        spikes |= 1u << w;
        s_spk[tid] = spikes;
      }
      xq_next[tid] = xq * a.beta_minus;
      const uint64_t mask = __ballot(spike);
      if (lane == w) my_mask = mask;
      if (lane == 0 && i / kWave < a.words) a.raster[(size_t)ring * a.words + i / kWave] = mask;
      ring = ring + 1 == a.raster_cap ? 0 : ring + 1;
    }
    lds_barrier();
    // ---- delivery of the next step's arrivals, and their depression ----
    const uint32_t m = w + 1, cnt = s_pre[m + 1] - s_pre[m];
    const bool ltd = m < steps || !a.last;
    uint32_t more = 0, direct = 0;  // bit u: what sub-row u has left to do
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      if (u * rows < cnt) {  // uniform
        if (ahead.len[u] > lanes) (ahead.len[u] == kDirect ? direct : more) |= 1u << u;
        if (sub < ahead.len[u] && ahead.len[u] != kDirect) {
          const uint32_t x = ahead.x[u] & (kPlasticTarget - 1u);
          const bool plastic = ahead.x[u] & kPlasticTarget;
          const float wv = ahead.w[u];
          float nw = wv;
          const uint32_t pend = s_spk[x] >> ahead.from[u] << ahead.from[u];
          if (plastic && pend) nw = potentiate(a, hdr[s_pre[m] + f_first + u * rows].trace, pend, nw);
          atomicAdd(&acc[x], __float2int_rn(nw * 65536.0f));
          const float dw = a.a_minus * xq_next[x];
          float lw = nw - dw;
          if (lw < 0.0f) lw = 0.0f;
          if (plastic && ltd) nw = lw;
          if (__float_as_uint(nw) != __float_as_uint(wv)) a.w_f32[ahead.e[u]] = nw;
        }
      }
    }
    if (cnt > kU * rows || __any((int)(more | direct))) {
      uint32_t u = 0;
      for (uint32_t f = f_first; f < cnt; f += rows, ++u) {
        const bool all = u >= kU || ((direct >> u) & 1u);
        if (all || ((more >> u) & 1u)) general(m, f, all ? sub : sub + lanes);
      }
    }
    if (m < steps) fetch(m + 1);
    if (any_again) __syncthreads();
    else lds_barrier();
  }
  if (active) {
    a.v[i] = v;
    a.ref[i] = ref;
    a.input[i] = acc[tid];
    a.x_pre[i] = xp;
    a.x_post[i] = xq;
  }

  // ---- the spikes: into the lists of their steps, and for the potentiation still due ----
  const bool due = spikes != 0 && in_len != 0;
  const uint64_t dues = __ballot(due);
  if (lane < steps) s_base[wave][lane] = (uint32_t)__popcll(my_mask);
  if (lane == 0) s_base[wave][kPlasticSteps] = (uint32_t)__popcll(dues);
  __syncthreads();
  if (tid < steps || tid == kPlasticSteps) {
    uint32_t sum = 0;
#pragma unroll
    for (int u = 0; u < kWaves; ++u) {
      const uint32_t c = s_base[u][tid];
      s_base[u][tid] = sum;
      sum += c;
    }
    uint32_t *counter = tid < steps ? list_count(t0 + tid, a) : a.ltp_len[a.parity];
    const uint32_t base = sum ? atomicAdd(counter, sum) : 0u;
#pragma unroll
    for (int u = 0; u < kWaves; ++u) s_base[u][tid] += base;
  }
  __syncthreads();
  for (uint32_t w = 0; w < steps; ++w) {
    const uint64_t mask = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(my_mask >> 32), (int)w) << 32) |
                          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)my_mask, (int)w);
    if ((spikes >> w) & 1u) list_ids(t0 + w, a)[s_base[wave][w] + lanes_below(mask)] = (int32_t)i;
  }
  if (due) {
    a.ltp[a.parity][s_base[wave][kPlasticSteps] + lanes_below(dues)] = make_uint4(in_lo, in_len, spikes, 0u);
    touched += (uint64_t)in_len * (uint32_t)__popc(spikes);
  }

  events = wave_sum(events);
  touched = wave_sum(touched);
  if (lane == 0) {
    const uint32_t part = ((r * kWaves + wave) % kCounterParts) * kLineU64;
    if (events) atomicAdd((unsigned long long *)&a.ctl->events[part], (unsigned long long)events);
    if (touched) atomicAdd((unsigned long long *)&a.ctl->touches[part], (unsigned long long)touched);
    if (r == 0 && wave == 0) {
      const uint32_t delivered = s_pre[steps + 1] - s_pre[1];
      if (delivered) atomicAdd((unsigned long long *)&a.ctl->spikes[0], (unsigned long long)delivered);
      // the next step's queue, and the step itself (this launch reads t_deliver)
      const uint32_t next = (uint32_t)((t0 + steps) % a.slots);
      for (uint32_t g = 0; g < kQueueGroups; ++g) a.q.qlen[(size_t)(next * kQueueGroups + g) * kQlenStride] = 0u;
      a.ctl->t = t0 + steps;
    }
  }
}

// Workgroup m: the list of the spikes of step t - 1 - m (t the step reached).
__global__ __launch_bounds__(kListBlock) void k_plastic_import(PlasticArgs a) {
  __shared__ uint32_t s_n;
  const uint64_t t = a.ctl->t;
  const uint64_t back = (uint64_t)blockIdx.x + 1;
  if (t < back) return;
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  const uint64_t *row = raster_row(t - back, a);
  int32_t *ids = list_ids(t - back, a);
  for (uint32_t x = threadIdx.x; x < a.words; x += kListBlock) {
    const uint64_t bits = row[x];
    if (!bits) continue;
    uint32_t p = atomicAdd(&s_n, (uint32_t)__popcll(bits));
    for (uint64_t b = bits; b; b &= b - 1) ids[p++] = (int32_t)(x * kWave + (uint32_t)__builtin_ctzll(b));
  }
  __syncthreads();
  if (threadIdx.x == 0) *list_count(t - back, a) = s_n;
}

// Workgroup m: the queue of step t - 1 - m (t the step reached), every spike in the
// sub-queue where the neuron update would append it.
__global__ __launch_bounds__(kListBlock) void k_plastic_export(PlasticArgs a) {
  __shared__ uint32_t s_len[kQueueGroups];
  const uint64_t t = a.ctl->t;
  const uint64_t back = (uint64_t)blockIdx.x + 1;
  if (t < back) return;
  const uint64_t s = t - back;
  const uint32_t slot = (uint32_t)(s % a.slots);
  if (threadIdx.x < kQueueGroups) s_len[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t *row = raster_row(s, a);
  for (uint32_t x = threadIdx.x; x < a.words; x += kListBlock) {
    const uint64_t bits = row[x];
    if (!bits) continue;
    const uint32_t g = x * kWave / kUpdateBlock % kQueueGroups;
    uint32_t p = atomicAdd(&s_len[g], (uint32_t)__popcll(bits));
    for (uint64_t b = bits; b; b &= b - 1, ++p)
      if (p < a.q.group_cap)
        a.q.ids[(size_t)slot * a.q.stride + g * a.q.group_cap + p] = (int32_t)(x * kWave + (uint32_t)__builtin_ctzll(b));
  }
  __syncthreads();
  if (threadIdx.x < kQueueGroups)
    a.q.qlen[(size_t)(slot * kQueueGroups + threadIdx.x) * kQlenStride] = s_len[threadIdx.x];
}

}  // namespace

hipError_t launch_plastic_import(const PlasticArgs &a, hipStream_t s) {
  k_plastic_import<<<a.delay, kListBlock, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_plastic_window(const PlasticArgs &a, uint32_t steps, hipStream_t s) {
  if (steps == 0 || steps >= a.delay || steps > kPlasticSteps || a.range == 0 || a.range > kPlasticBlock ||
      a.range % kWave != 0 || (uint64_t)a.ranges * a.range < a.n || a.raster_cap <= a.delay ||
      a.row_cap > kPlasticRows || a.row_blocks == 0 || a.list_slots < a.delay + steps + 1)
    return hipErrorInvalidValue;
  k_plastic_prepare<<<a.ltp_blocks + a.row_blocks + (a.n + kPrepBlock - 1) / kPrepBlock, kPrepBlock, 0, s>>>(a, steps);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_plastic_window<<<(a.ranges + kXcds - 1) / kXcds * kXcds, kPlasticBlock, 0, s>>>(a, steps);
  return hipGetLastError();
}

hipError_t launch_plastic_export(const PlasticArgs &a, hipStream_t s) {
  k_plastic_prepare<<<a.ltp_blocks, kPrepBlock, 0, s>>>(a, 0);  // the potentiation left
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the slot of the step reached is behind these: the last window cleared it
  k_plastic_export<<<a.slots - 1, kListBlock, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace snn
