// batch.hip -- static networks stepped by one persistent launch: many independent ones (the
// batched form), or a small one by itself.
//
// Every workgroup owns one network for the whole launch and runs the step pipeline of
// Fig. 1 for it step after step, with nothing shared between workgroups:
//   * V and the refractory times live in registers (kPer neurons per lane; a wavefront
//     owns consecutive 64-neuron raster words);
//   * the delay ring of Q16 input accumulators ([delay][n] int32) lives in LDS, so
//     Receive Spikes is an LDS atomic add per synaptic event and the CSR rows are the
//     only HBM stream, read as 16-byte groups of 4 targets, several per lane in flight;
//   * the step's spike queue is compacted with one ballot per 64 neurons and one LDS
//     counter reservation per ballot that holds a spike, into LDS (entries past its
//     capacity go to the network's queue buffer);
//   * where the LDS has room, the row offsets are staged there as well;
//   * two workgroup barriers per step separate update, delivery and the next update; a
//     step without spikes needs only the first.
// The launch starts from, and (when `commit` is set) leaves, each network's state in
// the network's own buffers with the same layout the single-network pipeline uses, so
// both pipelines and every reader agree on a network's state between launches.
//
// Bound: a network's steps are a serial chain on one compute unit.  For large networks the
// update's vector instructions come first, so what concerns a spike (reset, refractory time,
// raster bit, queue) sits behind wave-uniform branches that few groups of words take, and a
// word costs eight; then the latency of a spike's row (bounds, targets).  A step of the
// largest of 96 networks (20,000 neurons) went from 7.9 to 3.4 us, of 512 from 8.6 to 5.2,
// against a loop that handled every word's spikes in line and looked up each spike's row
// bounds after the barrier.  Sharing long rows between more lanes when few spikes are queued
// gained nothing (40,000 neurons: 6.6 against 6.4 us) and cost short rows 0.2 us.
#include <climits>
#include <type_traits>

#include "device_math.h"
#include "snn_internal.h"

namespace snn {
namespace {

// 16-byte groups of a row per lane per round: four, except in 1,024-thread workgroups
// (at most 128 registers per lane) where more would spill: two, and one where the drive's
// code also holds registers beside 16 or more neurons per lane.
constexpr int groups_in_flight(int block, int per, bool drive) {
  return block == 1024 ? (per >= 16 && drive ? 1 : 2) : 4;
}

// Words whose inputs are read together before their neurons are advanced.  A wavefront takes
// whole chunks of words.  Without a drive a word is little work and chunks of four or five cost
// nothing; with one it is a Philox block and a threshold search, and a chunk that leaves
// wavefronts of a small network without a word is a loss: in workgroups for up to 4,096 neurons a
// chunk is one word, up to 8,192 two.  256 driven networks of 300 neurons: 4.9 us a step with
// chunks of four, 2.6 with one; 300 of 1,000 neurons 10.8 and 6.7; 300 of 5,000 28.7 and 26.7
// (24.9 with one, which costs 300 of 8,000 2 %); 300 of 20,000 96.4, and 99.8 with one.
constexpr int update_chunk(int block, int per, bool drive) {
  return drive && block * per <= 4096 ? 1 : drive && block * per <= 8192 ? 2 : per % 5 == 0 ? 5 : 4;
}

// The value itself, as one that the compiler knows nothing about (uniform, per lane).
__device__ __forceinline__ uint32_t opaque(uint32_t x) {
  asm volatile("" : "+s"(x));
  return x;
}
__device__ __forceinline__ uint32_t opaque_lane(uint32_t x) {
  asm volatile("" : "+v"(x));
  return x;
}

// A queued spike: its neuron and the bounds of its row (a persistent network holds fewer than
// 2^32 synapses: at most 40,960^2).
struct QueuedRow {
  uint32_t src, lo, hi;
};

// LDS atomic adds of the elements [lo, hi) of one 16-byte group starting at edge e0.
__device__ __forceinline__ void add_group(int32_t *in, const int4 &c, const int4 &w, uint32_t e0, uint32_t lo,
                                          uint32_t hi) {
  const int32_t cv[4] = {c.x, c.y, c.z, c.w}, wv[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (e0 + q >= lo && e0 + q < hi) atomicAdd(&in[cv[q]], wv[q]);
}

template <int kBlock, int kPer, bool kDrive>
__device__ __forceinline__ void step_network(const BatchNet &d, uint32_t steps, uint32_t flags, LdsPlan lds) {
  // [delay][n] accumulators, the drive thresholds, q_cap queue entries, then, where they
  // fit, the n + 1 row offsets
  extern __shared__ int32_t s_dyn[];
  __shared__ uint32_t s_qn[3];
  __shared__ uint32_t s_group[kQueueGroups];
  __shared__ unsigned long long s_count[2];

  constexpr int kWaves = kBlock / kWave;
  constexpr int kChunk = update_chunk(kBlock, kPer, kDrive);
  constexpr int kGroupsInFlight = groups_in_flight(kBlock, kPer, kDrive);
  // a wavefront's words are stepped in spans of at most 64: a bit of `fired` and a raster
  // lane per word
  constexpr int kSpan = kPer <= kWave ? kPer : kPer / 2;
  using Bits = std::conditional_t<(kSpan > 32), uint64_t, uint32_t>;
  static_assert(kSpan % kChunk == 0 && kPer % kSpan == 0 && kSpan <= kWave, "whole chunks per span");
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const uint32_t n = d.n, delay = d.delay, q_cap = lds.q_cap;
  int32_t *acc = s_dyn;
  uint32_t *tbl = reinterpret_cast<uint32_t *>(s_dyn + (size_t)delay * n);
  QueuedRow *s_queue = reinterpret_cast<QueuedRow *>(tbl + d.below);
  uint32_t *s_row = reinterpret_cast<uint32_t *>(s_queue + q_cap);
  const bool rows_in_lds = delay * n + d.below + 3u * q_cap + n + 1u <= lds.words;
  const uint64_t t0 = d.ctl->t;

  // this wavefront's words [w0, w0 + per), whole chunks of them; neuron i0 + 64 k in lane `lane` of word k
  const uint32_t per = (d.words + kWaves * kChunk - 1) / (kWaves * kChunk) * kChunk;
  const uint32_t w0 = wave * per, i0 = w0 * kWave + lane;
  // Refractory until step `until` of this launch (exclusive): a spike at step s sets it to
  // s + 1 + ref_steps, so that no counter has to be decremented; lanes past n are
  // refractory for good.
  float v[kPer];
  int32_t until[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const uint32_t i = i0 + (uint32_t)k * kWave;
    const bool mine = (uint32_t)k < per && i < n;
    v[k] = mine ? d.v[i] : 0.f;
    until[k] = mine ? d.ref[i] : INT_MAX;
  }
  const uint32_t n_acc = delay * n;
  for (uint32_t j0 = tid; j0 < n_acc; j0 += 8 * kBlock) {  // eight loads in flight
    int32_t x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t j = j0 + (uint32_t)u * kBlock;
      x[u] = j < n_acc ? d.input[j] : 0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t j = j0 + (uint32_t)u * kBlock;
      if (j < n_acc) acc[j] = x[u];
    }
  }
  if (kDrive)
    for (uint32_t j = tid; j < d.below; j += kBlock) tbl[j] = d.table32[j];
  if (rows_in_lds)
    for (uint32_t j = tid; j <= n; j += kBlock) s_row[j] = (uint32_t)d.row_ptr[j];
  if (tid < 3) s_qn[tid] = 0;
  if (tid < 2) s_count[tid] = 0;
  if (tid < kQueueGroups) s_group[tid] = 0;
  __syncthreads();

  const uint32_t shift = d.lanes_shift;
  const uint32_t lanes = 1u << shift, groups = kBlock >> shift;
  const uint32_t grp = tid >> shift, gl = tid & (lanes - 1u);
  const bool write_raster = (flags & kBatchWriteRaster) != 0;
  // the steps whose queues the FIFO ring still holds after this launch
  const uint32_t ring_from = (flags & kBatchQueues) ? (steps > d.slots ? steps - d.slots : 0u) : steps;
  uint32_t slot = (uint32_t)(t0 % delay);
  uint32_t ras = (uint32_t)(t0 % d.raster_cap);
  uint32_t qslot = (uint32_t)(t0 % d.slots);
  uint32_t qi = 0;  // s mod 3
  uint64_t events = 0, spikes = 0;

  // the drive's share of a neuron's input of step t (a refractory neuron discards it)
  auto advance_input = [&](int32_t x, bool refractory, uint32_t i, uint64_t t) -> int32_t {
    if (!kDrive) return x;
    if (d.below == 0 || refractory) return x;
    const Words4 r4 = philox(i, (uint32_t)(t >> 2), (uint32_t)(t >> 34), kStreamPoisson, d.key0, d.key1);
    const uint32_t r = word_of(r4, (uint32_t)t & 3u);
    uint32_t kk = 0;
    while (kk < d.below && tbl[kk] <= r) ++kk;
    return (int32_t)((uint32_t)x + kk * (uint32_t)d.w_ext_q16);
  };
  // V and the refractory times have arrived: without this wait the compiler waits in every
  // step, for the previous step's raster stores too
  __builtin_amdgcn_s_waitcnt(0);

  for (uint32_t s = 0; s < steps; ++s) {
    const uint64_t t = t0 + s;
    int32_t *in = acc + (size_t)slot * n;
    uint32_t *qn = &s_qn[qi];
    const uint32_t qnext = qslot + 1u == d.slots ? 0u : qslot + 1u;
    int32_t *spill = d.queue + (size_t)qnext * d.queue_stride;  // queue entries past q_cap
    const bool ring = s >= ring_from;
    // (the opaque copies keep what depends on n and i0 from being computed once for every
    // word ahead of the loop and held in registers)
    const uint32_t n_s = opaque(n), i0_s = opaque_lane(i0);
    // ---- Update Neurons: step t for every neuron of the network ----
    uint64_t words[kPer / kSpan];  // per span, lane k: its raster word k
#pragma unroll
    for (int span = 0; span < kPer; span += kSpan) {
      Bits fired = 0;     // bit k: this lane's neuron of the span's word k spikes
      uint64_t word = 0;  // lane k: the span's raster word k
#pragma unroll
      for (int k0 = span; k0 < span + kSpan; k0 += kChunk) {
        if ((uint32_t)k0 < per) {  // uniform
          int32_t x[kChunk];
          if ((w0 + (uint32_t)(k0 + kChunk)) * kWave <= n_s) {  // uniform: every lane has a neuron
#pragma unroll
            for (int u = 0; u < kChunk; ++u) x[u] = in[i0_s + (uint32_t)(k0 + u) * kWave];
#pragma unroll
            for (int u = 0; u < kChunk; ++u) in[i0_s + (uint32_t)(k0 + u) * kWave] = 0;
          } else {
#pragma unroll
            for (int u = 0; u < kChunk; ++u) {
              const uint32_t i = i0_s + (uint32_t)(k0 + u) * kWave;
              x[u] = 0;
              if (i < n_s) {
                x[u] = in[i];
                in[i] = 0;
              }
            }
          }
#pragma unroll
          for (int u = 0; u < kChunk; ++u) x[u] = advance_input(x[u], until[k0 + u] > (int32_t)s, i0_s + (uint32_t)(k0 + u) * kWave, t);
          uint64_t mask[kChunk], some = 0;
#pragma unroll
          for (int u = 0; u < kChunk; ++u) {
            const int k = k0 + u;
            const bool refractory = until[k] > (int32_t)s;
            // lif_advance's operations; V + input 2^-16 as one fused operation, which rounds
            // the same because the product is exact
            float vv = __builtin_fmaf((float)x[u], 0x1p-16f, v[k]);
            const float diff = vv - d.v_inf;
            const float leak = diff * d.alpha;
            vv = d.v_inf + leak;
            mask[u] = __builtin_amdgcn_ballot_w64(vv >= d.v_th) & ~__builtin_amdgcn_ballot_w64(refractory);
            v[k] = refractory ? v[k] : vv;
            some |= mask[u];
          }
          if (__builtin_expect(some != 0, 0)) {  // uniform
#pragma unroll
            for (int u = 0; u < kChunk; ++u) {
              const int k = k0 + u;
              if (__builtin_amdgcn_inverse_ballot_w64(mask[u])) {
                v[k] = d.v_reset;
                until[k] = (int32_t)s + 1 + d.ref_steps;
                fired |= (Bits)1 << (k - span);
              }
            }
          }
        }
      }
      const uint32_t ws0 = w0 + span, is0 = i0_s + span * kWave;
      if (__ballot(fired != 0)) {  // uniform
        // one reservation for the wavefront's spikes of this span; every lane queues its own
        // with their row's bounds, so that the delivery starts from the rows
        const uint32_t mine = (uint32_t)__popcll((uint64_t)fired);
        const uint32_t incl = wave_inclusive_scan(mine);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(qn, total);
        // meanwhile the raster words that hold spikes, one by one
        Bits left = fired;
        for (uint64_t any = __ballot(left != 0); any; any = __ballot(left != 0)) {
          const uint32_t first = (uint32_t)__builtin_ctzll(any);
          uint64_t one = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)left, (int)first);
          if (kSpan > 32)
            one |= (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)left >> 32), (int)first) << 32;
          const uint32_t k = (uint32_t)__builtin_ctzll(one);  // uniform
          const bool spike = (left >> k) & 1u;
          const uint64_t mask = __ballot(spike);
          left &= ~((Bits)1 << k);
          if (lane == k) word = mask;
          if (ring) {  // the step's queue as the single-network pipeline lays it out
            const uint32_t g = ((ws0 + k) / (kUpdateBlock / kWave)) % kQueueGroups;
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&s_group[g], (uint32_t)__popcll(mask));
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + lanes_below(mask);
            if (spike && at < d.group_cap)
              d.queue[(size_t)qslot * d.queue_stride + g * d.group_cap + at] = (int32_t)(is0 + k * kWave);
          }
        }
        uint32_t pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + incl - mine;
        for (; fired; fired &= fired - 1, ++pos) {
          const uint32_t i = is0 + (uint32_t)__builtin_ctzll((uint64_t)fired) * kWave;
          if (pos < q_cap) {
            QueuedRow r{i, 0, 0};
            if (rows_in_lds) {
              r.lo = s_row[i];
              r.hi = s_row[i + 1u];
            } else {
              r.lo = (uint32_t)d.row_ptr[i];
              r.hi = (uint32_t)d.row_ptr[i + 1u];
            }
            s_queue[pos] = r;
          } else {
            spill[pos - q_cap] = (int32_t)i;
          }
        }
      }
      words[span / kSpan] = word;
    }
    __syncthreads();
    // ---- Receive Spikes: S_t into the accumulator of arrival step t + delay, which
    //      is slot t mod delay again (read and cleared above) ----
    // (the group's first queue entry is read along with the count)
    const QueuedRow ahead = s_queue[grp < q_cap ? grp : 0u];
    const uint32_t count = (uint32_t)__builtin_amdgcn_readfirstlane((int)*qn);  // uniform
    // The counter of step s + 2 was last read before this step's barrier and is next used
    // after step s + 1's.
    if (tid == 0) s_qn[qi == 0 ? 2 : qi - 1] = 0;
    if (ring && tid < kQueueGroups) {
      d.qlen[(size_t)(qslot * kQueueGroups + tid) * kQlenStride] = s_group[tid];
      s_group[tid] = 0;
    }
    if (count) {
      for (uint32_t q = grp; q < count; q += groups) {
        QueuedRow r = ahead;
        if (q != grp || grp >= q_cap) {
          if (q < q_cap) {
            r = s_queue[q];
          } else {
            r.src = (uint32_t)spill[q - q_cap];
            r.lo = (uint32_t)d.row_ptr[r.src];
            r.hi = (uint32_t)d.row_ptr[r.src + 1u];
          }
        }
        const uint32_t lo = r.lo, hi = r.hi;
        const int32_t ws = d.w_src ? d.w_src[r.src] : 0;  // one weight per source: targets only
        if (gl == 0) {
          events += hi - lo;
          spikes += 1;
        }
        // the row as 16-byte groups of 4 targets (the arrays are padded to whole groups),
        // up to kGroupsInFlight groups per lane requested before their adds; elements
        // outside the row are masked
        const uint32_t g_lo = lo >> 2, g_hi = (uint32_t)(((uint64_t)hi + 3) >> 2);
        const int4 *col4 = reinterpret_cast<const int4 *>(d.col);
        const int4 *w4 = reinterpret_cast<const int4 *>(d.w_q16);
        for (uint32_t g0 = g_lo + gl; g0 < g_hi; g0 += kGroupsInFlight * lanes) {
          int4 c[kGroupsInFlight], w[kGroupsInFlight];
#pragma unroll
          for (int u = 0; u < kGroupsInFlight; ++u) {
            const uint32_t g = g0 + (uint32_t)u * lanes;
            c[u] = g < g_hi ? col4[g] : make_int4(0, 0, 0, 0);
            w[u] = make_int4(ws, ws, ws, ws);
            if (!d.w_src && g < g_hi) w[u] = w4[g];
          }
#pragma unroll
          for (int u = 0; u < kGroupsInFlight; ++u) {
            const uint32_t g = g0 + (uint32_t)u * lanes;
            if (g < g_hi) add_group(in, c[u], w[u], 4u * g, lo, hi);
          }
        }
      }
    }
    // after the delivery's loads, which would otherwise wait for these stores
    if (write_raster) {
#pragma unroll
      for (int h = 0; h < kPer / kSpan; ++h) {
        const uint32_t w = (uint32_t)h * kSpan + lane;
        if (lane < kSpan && w < per && w0 + w < d.words) d.raster[(size_t)ras * d.words + w0 + w] = words[h];
      }
    }
    if (count || ring) __syncthreads();
    slot = slot + 1u == delay ? 0u : slot + 1u;
    ras = ras + 1u == d.raster_cap ? 0u : ras + 1u;
    qslot = qnext;
    qi = qi == 2 ? 0 : qi + 1;
  }

  if (!(flags & kBatchCommit)) return;
  const uint32_t n_e = opaque(n), i0_e = opaque_lane(i0);
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const uint32_t i = i0_e + (uint32_t)k * kWave;
    if ((uint32_t)k < per && i < n_e) {
      d.v[i] = v[k];
      // a count that was not positive stays as it was until the neuron spikes
      const int32_t r0 = d.ref[i], left = until[k] - (int32_t)steps;
      d.ref[i] = r0 <= 0 && until[k] == r0 ? r0 : (left > 0 ? left : 0);
    }
  }
  __syncthreads();  // a last step without spikes ends without a barrier
  for (uint32_t j = tid; j < n_acc; j += kBlock) d.input[j] = acc[j];
  if (flags & kBatchQueues)  // the next window's queues start empty
    for (uint32_t j = tid; j < d.window * kQueueGroups; j += kBlock)
      d.qlen[(size_t)((qslot + j / kQueueGroups) % d.slots * kQueueGroups + j % kQueueGroups) * kQlenStride] = 0;
  events = wave_sum(events);
  spikes = wave_sum(spikes);
  if (lane == 0) {
    if (events) atomicAdd(&s_count[0], (unsigned long long)events);
    if (spikes) atomicAdd(&s_count[1], (unsigned long long)spikes);
  }
  __syncthreads();
  if (tid == 0) {
    d.ctl->events[0] += s_count[0];
    d.ctl->spikes[0] += s_count[1];
    d.ctl->t = t0 + steps;
  }
}

template <int kBlock, int kPer, bool kDrive>
__global__ __launch_bounds__(kBlock) void k_batch(const BatchNet *nets, const uint32_t *order,
                                                  uint32_t steps, uint32_t flags, LdsPlan lds) {
  const BatchNet d = nets[order[blockIdx.x]];
  step_network<kBlock, kPer, kDrive>(d, steps, flags, lds);
}

// One network by itself, its description in the kernel's arguments.
template <int kBlock, int kPer, bool kDrive>
__global__ __launch_bounds__(kBlock) void k_solo(BatchNet d, uint32_t steps, uint32_t flags, LdsPlan lds) {
  step_network<kBlock, kPer, kDrive>(d, steps, flags, lds);
}

template <int kBlock, int kPer>
hipError_t launch_one(const BatchNet *nets, const uint32_t *order, uint32_t n_nets, uint32_t steps,
                      uint32_t flags, LdsPlan lds, hipStream_t s) {
  // without a Poisson drive in any member the kernel is built without the drive's code
  // (Philox and the threshold scan), which would otherwise take registers
  auto k = (flags & kBatchDrive) ? k_batch<kBlock, kPer, true> : k_batch<kBlock, kPer, false>;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds.words * 4);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(n_nets), dim3(kBlock), (size_t)lds.words * 4, s, nets, order, steps, flags, lds);
  return hipGetLastError();
}

template <int kBlock, int kPer>
hipError_t launch_solo_one(const BatchNet &d, uint32_t steps, uint32_t flags, LdsPlan lds, hipStream_t s) {
  auto k = k_solo<kBlock, kPer, false>;
  if (lds.words > 16384) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds.words * 4);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k, dim3(1), dim3(kBlock), (size_t)lds.words * 4, s, d, steps, flags, lds);
  return hipGetLastError();
}

}  // namespace

bool batch_variant_supported(uint32_t block, uint32_t per) {
  switch (block) {
    case 256: return per == 16 || per == 32 || per == 64 || per == 80;
    case 512: return per == 8 || per == 16 || per == 32 || per == 40;
    case 1024: return per == 4 || per == 8 || per == 16 || per == 20;
    default: return false;
  }
}

uint32_t batch_per_lane(uint32_t block, uint32_t n_max) {
  const uint32_t need = (n_max + block - 1) / block;
  static const uint32_t k256[] = {16, 32, 64, 80}, k512[] = {8, 16, 32, 40}, k1024[] = {4, 8, 16, 20};
  const uint32_t *opts = block == 256 ? k256 : block == 512 ? k512 : k1024;
  for (int j = 0; j < 4; ++j)
    if (opts[j] >= need) return opts[j];
  return 0;
}

hipError_t launch_batch(const BatchNet *nets, const uint32_t *order, uint32_t n_nets, uint32_t steps,
                        uint32_t block, uint32_t per, uint32_t flags, LdsPlan lds, hipStream_t s) {
#define SNN_BATCH_CASE(B, K) \
  if (block == B && per == K) return launch_one<B, K>(nets, order, n_nets, steps, flags, lds, s);
  SNN_BATCH_CASE(256, 16) SNN_BATCH_CASE(256, 32) SNN_BATCH_CASE(256, 64) SNN_BATCH_CASE(256, 80)
  SNN_BATCH_CASE(512, 8) SNN_BATCH_CASE(512, 16) SNN_BATCH_CASE(512, 32) SNN_BATCH_CASE(512, 40)
  SNN_BATCH_CASE(1024, 4) SNN_BATCH_CASE(1024, 8) SNN_BATCH_CASE(1024, 16) SNN_BATCH_CASE(1024, 20)
#undef SNN_BATCH_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_solo(const BatchNet &d, uint32_t steps, uint32_t flags, LdsPlan lds, hipStream_t s) {
  // the smallest number of neurons per lane: at 1,000 neurons 256 threads step in 0.87 us
  // (1,024 in 0.99), at 4,000 neurons 1,024 threads in 1.40 us (512 in 1.60)
  if (d.n <= 256 * 4) return launch_solo_one<256, 4>(d, steps, flags, lds, s);
  if (d.n <= 1024 * 4) return launch_solo_one<1024, 4>(d, steps, flags, lds, s);
  if (d.n <= 1024 * 8) return launch_solo_one<1024, 8>(d, steps, flags, lds, s);
  if (d.n <= 1024 * 20) return launch_solo_one<1024, 20>(d, steps, flags, lds, s);
  if (d.n <= kSoloMaxNeurons) return launch_solo_one<1024, 40>(d, steps, flags, lds, s);
  return hipErrorInvalidValue;
}

}  // namespace snn
