// bptt.hip -- surrogate-gradient BPTT of a recurrent LIF network with sparse input and
// recurrent weights (CSR, FP32) and a dense leaky readout: forward pass and hand-written
// adjoint.
//
// Layouts (batch innermost, so that one wavefront = 64 batch elements of one neuron and
// every gather of a presynaptic value is one coalesced 256-byte row):
//   xt    [T][n_in][64]      input spikes (transposed from the caller's [B][T][n_in])
//   s     [T][H][64]         hidden outputs of every step
//   vck   [T/K][H][64]       membrane potential before each checkpoint segment
//   vseg  [K][H][64]         membranes of one segment, recomputed in the backward pass
//   lamu  [T][O][64]         readout adjoint
//   lamv  [T][S][H][8]       membrane adjoint of every step, in S slices of 8 batch elements
//                            ([T][H][64] without slices; + zeros for step T)
//   xbits [C][T], sbits [H][T]  64-bit batch masks of the binary input and hidden spikes
//                            (8 readable entries after each, and before sbits)
// Weights stay in the caller's CSR order (rows = presynaptic neuron, sorted targets);
// the forward current is a gather over the transposed index (per target, sources in
// ascending order, input projection first), the adjoint's dL/ds a gather over the
// forward rows, and every weight gradient has exactly one owner.
#include <algorithm>

#include "device_math.h"
#include "snn_internal.h"

namespace snn {
namespace {

__device__ __forceinline__ float spike_fn(float z, float slope, bool smooth) {
  if (smooth) {
    const float a = slope * z;
    const float d = 1.0f + fabsf(a);
    return 0.5f + 0.5f * (a / d);
  }
  return z >= 0.0f ? 1.0f : 0.0f;
}

__device__ __forceinline__ float surrogate(float z, float slope, bool smooth) {
  const float d = 1.0f + slope * fabsf(z);
  const float g = 1.0f / (d * d);
  return smooth ? 0.5f * slope * g : g;
}

__device__ __forceinline__ bool finite_f32(float x) { return (__float_as_uint(x) & 0x7f800000u) != 0x7f800000u; }

// Where the plan takes slices (BpttArgs::S) the membrane adjoint is held in slices of 8
// batch elements, lamv[t][slice][H][8], of which there are S = ceil(B / 8).
__device__ __forceinline__ size_t slice_index(const BpttArgs &a, uint32_t t, uint32_t b, uint32_t j) {
  return (((size_t)t * a.S + (b >> 3)) * a.H + j) * 8 + (b & 7u);
}

// x [B][T][C] -> xt [T][C][64]; lanes >= B hold zeros.  A workgroup per (step t, block of
// 64 inputs) reads the 64 batch rows of its block (256 bytes each, coalesced) into LDS and
// writes the block transposed; a wavefront per input c then also writes that input's
// batch mask xbits[c][t] (bit b: x != 0) and sets flags[0] if some value is neither 0 nor 1
// (k_bits' rule).  Beside that the grid looks over n_out readout weights and sets flags[2] if some
// are not finite: here the look costs nothing (6.5 us at 19 x 103 x 77 with and without it; 3 us
// with 360,000 weights), in k_input_current_values, which otherwise returns at once, 0.7 us.
__global__ __launch_bounds__(256) void k_transpose_x(const float *x, float *xt, uint64_t *xbits, uint32_t *flags,
                                                     uint32_t B, uint32_t T, uint32_t C, const float *w_out,
                                                     uint32_t n_out) {
  __shared__ float tile[64][65];
  const uint32_t t = blockIdx.y, c0 = blockIdx.x * 64u;
  const uint32_t l = threadIdx.x % 64u, r = threadIdx.x / 64u;
  for (uint32_t b = r; b < 64u; b += 4u)
    tile[b][l] = b < B && c0 + l < C ? x[((uint64_t)b * T + t) * C + c0 + l] : 0.0f;
  __syncthreads();
  for (uint32_t k = r; k < 64u && c0 + k < C; k += 4u) {
    const uint32_t c = c0 + k;
    const float v = tile[l][k];
    xt[((uint64_t)t * C + c) * 64u + l] = v;
    const bool on = l < B && v != 0.0f;
    const uint64_t m = __ballot(on);
    const uint64_t bad = __ballot(on && v != 1.0f);
    if (l == 0) {
      xbits[(size_t)c * T + t] = m;
      if (bad) atomicOr(flags, 1u);
    }
  }
  bool finite = true;
#pragma unroll 8
  for (uint32_t e = (t * gridDim.x + blockIdx.x) * 256u + threadIdx.x; e < n_out; e += gridDim.x * T * 256u)
    finite &= finite_f32(w_out[e]);
  if (!finite) atomicOr(flags + 2, 1u);
}

// Transposed-order copy of a CSR weight vector: w_t[e] = w[edge[e]].
__global__ void k_gather_t(const float *w, const uint32_t *edge, float *w_t, uint64_t nnz) {
  const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < nnz) w_t[e] = w[edge[e]];
}

// sum += w[e] * val[src[e] * 64 + b] over [e0, e1), one term at a time in edge order.
// The (wave-uniform) sources and weights of the next kChunk edges are fetched while the
// presynaptic values of the current chunk are in flight, so each chunk costs about one
// memory round trip.
constexpr int kChunk = 16;
__device__ __forceinline__ float ordered_gather_sum(float acc, uint64_t e0, uint64_t e1, const int32_t *src,
                                                    const float *w, const float *val, uint32_t b) {
  uint64_t e = e0;
  int32_t sr[kChunk];
  float wv[kChunk];
  if (e + kChunk <= e1) {
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      sr[u] = src[e + u];
      wv[u] = w[e + u];
    }
  }
  while (e + kChunk <= e1) {
    float xv[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) xv[u] = val[(size_t)sr[u] * 64 + b];
    int32_t sn[kChunk];
    float wn[kChunk];
    const bool more = e + 2 * kChunk <= e1;
    if (more) {
#pragma unroll
      for (int u = 0; u < kChunk; ++u) {
        sn[u] = src[e + kChunk + u];
        wn[u] = w[e + kChunk + u];
      }
    }
#pragma unroll
    for (int u = 0; u < kChunk; ++u) acc = acc + wv[u] * xv[u];
    if (more) {
#pragma unroll
      for (int u = 0; u < kChunk; ++u) {
        sr[u] = sn[u];
        wv[u] = wn[u];
      }
    }
    e += kChunk;
  }
  for (; e < e1; ++e) acc = acc + w[e] * val[(size_t)src[e] * 64 + b];
  return acc;
}

// The same ordered sum with two chunks of presynaptic values in flight: the values of
// chunk c + 1 are requested before the terms of chunk c are added, so that a chunk costs
// about half a memory round trip.  For the per-step kernels, where one wavefront per
// neuron is all the parallelism a step has.
__device__ __forceinline__ float ordered_gather_pipe(float acc, uint64_t e0, uint64_t e1, const int32_t *src,
                                                     const float *w, const float *val, uint32_t b) {
  uint64_t e = e0;
  if (e + 2 * kChunk <= e1) {
    int32_t sa[kChunk], sb[kChunk];
    float wa[kChunk], wb[kChunk], xa[kChunk], xb[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      sa[u] = src[e + u];
      wa[u] = w[e + u];
    }
#pragma unroll
    for (int u = 0; u < kChunk; ++u) xa[u] = val[(size_t)sa[u] * 64 + b];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      sb[u] = src[e + kChunk + u];
      wb[u] = w[e + kChunk + u];
    }
    // invariant: chunk e is in (wa, xa), chunk e + kChunk (whole) has its sources in sb
    while (true) {
#pragma unroll
      for (int u = 0; u < kChunk; ++u) xb[u] = val[(size_t)sb[u] * 64 + b];
      const bool more = e + 3 * kChunk <= e1;
      if (more) {
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
          sa[u] = src[e + 2 * kChunk + u];
        }
      }
#pragma unroll
      for (int u = 0; u < kChunk; ++u) acc = acc + wa[u] * xa[u];
      e += kChunk;
      // chunk e is in (wb, xb)
#pragma unroll
      for (int u = 0; u < kChunk; ++u) {
        wa[u] = wb[u];
        xa[u] = xb[u];
      }
      if (!more) break;
#pragma unroll
      for (int u = 0; u < kChunk; ++u) {
        sb[u] = sa[u];
        wb[u] = w[e + kChunk + u];
      }
    }
#pragma unroll
    for (int u = 0; u < kChunk; ++u) acc = acc + wa[u] * xa[u];
    e += kChunk;
  }
  for (; e < e1; ++e) acc = acc + w[e] * val[(size_t)src[e] * 64 + b];
  return acc;
}

// The same ordered sum where every presynaptic value is 0 or 1, given as 64-bit batch
// masks: masks[src * stride + col] has bit b set where the value of batch element b is 1.
// A term then adds w[e] where the lane's bit is set and leaves the sum as it is where it
// is clear; that is the sum's own value, since w * 1 = w exactly and, for finite weights,
// adding w * 0 = +-0 leaves a sum that starts from +0 unchanged.  Lanes load the sources,
// weights and masks of 64 edges at once (two chunks, all requested before any term is
// added), and each edge's mask and weight reach the wavefront by lane reads, the mask as
// the lane condition: about two dependent memory round trips per 128 edges.
__device__ __forceinline__ uint64_t lane_read64(uint64_t x, uint32_t u) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, (int)u);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), (int)u);
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ float ordered_mask_sum(float acc, uint64_t e0, uint64_t e1, const int32_t *src,
                                                  const float *w, const uint64_t *masks, uint64_t stride,
                                                  uint32_t col) {
  const uint32_t l = lane_id();
  for (uint64_t base = e0; base < e1; base += 2u * kWave) {
    // loads from indices clamped to the last edge, issued unconditionally so that they
    // are all in flight together; the masks of lanes past e1 are then cleared
    const uint64_t last = e1 - 1;
    const uint64_t ea = std::min<uint64_t>(base + l, last), eb = std::min<uint64_t>(base + kWave + l, last);
    const uint32_t sa = (uint32_t)src[ea], sb = (uint32_t)src[eb];
    const float wa = w[ea], wb = w[eb];
    uint64_t ma = masks[(uint64_t)sa * stride + col];
    uint64_t mb = masks[(uint64_t)sb * stride + col];
    if (base + l >= e1) ma = 0u;
    if (base + kWave + l >= e1) mb = 0u;
    // edges past e1 carry an empty mask, so whole groups of eight run unconditionally
    const uint32_t na = (uint32_t)std::min<uint64_t>(e1 - base, kWave);
#pragma unroll 8
    for (uint32_t u = 0; u < ((na + 7u) & ~7u); ++u) {
      const float sum = acc + __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wa), (int)u));
      acc = __builtin_amdgcn_inverse_ballot_w64(lane_read64(ma, u)) ? sum : acc;
    }
    if (e1 - base > kWave) {
      const uint32_t nb = (uint32_t)std::min<uint64_t>(e1 - base - kWave, kWave);
#pragma unroll 8
      for (uint32_t u = 0; u < ((nb + 7u) & ~7u); ++u) {
        const float sum = acc + __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wb), (int)u));
        acc = __builtin_amdgcn_inverse_ballot_w64(lane_read64(mb, u)) ? sum : acc;
      }
    }
  }
  return acc;
}

// The ordered mask sums of kSteps consecutive columns at once (acc[u] for column
// col0 + u), for kernels with parallelism to spare: the edges are wave-uniform, so their
// sources, weights and each source's kSteps masks (contiguous in a row) arrive by scalar
// loads, and a mask serves directly as the lane condition.  A term costs one add and one
// select.  The masks of a group of edges and the sources of the next group are requested
// together.  Rows must hold kSteps - 1 readable entries past the last column used.
constexpr int kMaskSteps = 8;
constexpr int kMaskGroup = 4;
__device__ __forceinline__ void ordered_mask_sum_steps(float (&acc)[kMaskSteps], uint64_t e0, uint64_t e1,
                                                       const int32_t *src, const float *w,
                                                       const uint64_t *masks, uint64_t stride, int64_t col0) {
  uint64_t e = e0;
  if (e + kMaskGroup <= e1) {
    uint32_t c[kMaskGroup];
    float wv[kMaskGroup];
#pragma unroll
    for (int g = 0; g < kMaskGroup; ++g) {
      c[g] = (uint32_t)src[e + g];
      wv[g] = w[e + g];
    }
    while (true) {
      uint64_t mk[kMaskGroup][kMaskSteps];
#pragma unroll
      for (int g = 0; g < kMaskGroup; ++g) {
        const uint64_t *row = masks + (int64_t)((uint64_t)c[g] * stride) + col0;
#pragma unroll
        for (int u = 0; u < kMaskSteps; ++u) mk[g][u] = row[u];
      }
      float wc[kMaskGroup];
#pragma unroll
      for (int g = 0; g < kMaskGroup; ++g) wc[g] = wv[g];
      const bool more = e + 2 * kMaskGroup <= e1;
      if (more) {
#pragma unroll
        for (int g = 0; g < kMaskGroup; ++g) {
          c[g] = (uint32_t)src[e + kMaskGroup + g];
          wv[g] = w[e + kMaskGroup + g];
        }
      }
#pragma unroll
      for (int g = 0; g < kMaskGroup; ++g)
#pragma unroll
        for (int u = 0; u < kMaskSteps; ++u) {
          const float sum = acc[u] + wc[g];
          acc[u] = __builtin_amdgcn_inverse_ballot_w64(mk[g][u]) ? sum : acc[u];
        }
      e += kMaskGroup;
      if (!more) break;
    }
  }
  for (; e < e1; ++e) {
    const uint64_t *row = masks + (int64_t)((uint64_t)(uint32_t)src[e] * stride) + col0;
    const float wv = w[e];
#pragma unroll
    for (int u = 0; u < kMaskSteps; ++u) {
      const float sum = acc[u] + wv;
      acc[u] = __builtin_amdgcn_inverse_ballot_w64(row[u]) ? sum : acc[u];
    }
  }
}

// Input-projection current of every step: iin[t][j][b] = sum over j's input in-edges,
// sources ascending, from 0 -- the first part of the hidden current in its defined order.
// It does not depend on the recurrent state, so all steps run in parallel.  Two kernels,
// of which the flag that k_bits set for the inputs lets one work: with binary inputs
// (flags[0] clear) k_input_current takes the terms from the input masks, a wavefront per
// (block of kMaskSteps steps, j); otherwise k_input_current_values gathers the values,
// a wavefront per (t, j).
__global__ __launch_bounds__(256) void k_input_current(BpttArgs a) {
  if (a.flags[0] != 0) return;
  // wave-uniform index (readfirstlane lets the edge lists be read with scalar loads)
  const uint64_t w = (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t n_blocks = (a.T + kMaskSteps - 1) / kMaskSteps;
  if (w >= (uint64_t)n_blocks * a.H) return;
  const uint32_t t0 = (uint32_t)(w / a.H) * kMaskSteps, j = (uint32_t)(w % a.H);
  const uint32_t nt = std::min<uint32_t>(kMaskSteps, a.T - t0);
  const uint32_t b = lane_id();
  float acc[kMaskSteps];
#pragma unroll
  for (int u = 0; u < kMaskSteps; ++u) acc[u] = 0.0f;
  ordered_mask_sum_steps(acc, a.in_t_ptr[j], a.in_t_ptr[j + 1], a.in_t_src, a.w_in_t, a.xbits, a.T, t0);
#pragma unroll
  for (int u = 0; u < kMaskSteps; ++u) {
    if ((uint32_t)u >= nt) continue;
    if (!a.events) a.iin[((size_t)(t0 + u) * a.H + j) * 64 + b] = acc[u];
    else if (b < a.B) a.sg[slice_index(a, t0 + u, b, j)] = acc[u];  // the busy form
  }
}

// (a bounded grid that strides over the (t, j) pairs, so that the launch costs little
// when the flag sends it home.  An atomic before the sums would take their edge lists off the
// scalar unit: a forward pass of 64 x 250 x 700 -> 1,024 with inputs other than 0 and 1 took 4.5
// ms instead of 3.1.)
constexpr uint32_t kValuesGrid = 2048;
__global__ __launch_bounds__(256) void k_input_current_values(BpttArgs a, bool busy) {
  if (a.flags[0] == 0) return;
  const uint32_t b = lane_id();
  const uint64_t first = (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // the lane's place in vall, or of slice_index in sg for the busy form
  float *out = busy ? a.sg + slice_index(a, 0, b, 0) : a.vall + (size_t)b * a.Hp;
  const size_t step = busy ? (size_t)a.S * a.H * 8 : (size_t)a.B * a.Hp;
  const uint32_t neuron = busy ? 8 : 1;
  for (uint64_t w = first; w < (uint64_t)a.T * a.H; w += (uint64_t)gridDim.x * 4) {
    const uint32_t t = (uint32_t)(w / a.H), j = (uint32_t)(w % a.H);
    const float *xt = a.xt + (size_t)t * a.C * 64;
    if (!a.events) {
      a.iin[w * 64 + b] = ordered_gather_sum(0.0f, a.in_t_ptr[j], a.in_t_ptr[j + 1], a.in_t_src, a.w_in_t, xt, b);
      continue;
    }
    // the event-driven form holds the weights as dense rows; eight terms requested together
    float sum = 0.0f;
    const uint64_t e1 = a.in_t_ptr[j + 1];
    for (uint64_t e = a.in_t_ptr[j]; e < e1; e += 8) {
      float wv[8], x[8];
#pragma unroll
      for (uint32_t u = 0; u < 8; ++u) {
        const uint32_t c = (uint32_t)a.in_t_src[std::min<uint64_t>(e + u, e1 - 1)];
        wv[u] = a.dense_in[(size_t)c * a.Hp + j];
        x[u] = xt[(size_t)c * 64 + b];
      }
#pragma unroll
      for (uint32_t u = 0; u < 8; ++u)
        if (e + u < e1) sum = sum + wv[u] * x[u];
    }
    if (b < a.B) out[t * step + j * neuron] = sum;
  }
}

// One step t of the hidden layer: one wavefront per hidden neuron j, lane = batch.  The
// current continues the input part with j's recurrent in-edges (sources ascending).
// vprev/sprev are step t-1 (nullptr at t = 0).  Writes v_out[j][b] and, if s_out is
// set, s_out[j][b].  In spiking mode the spikes are 0 or 1: the recurrent terms come
// from the masks of step t-1, and the step writes its own masks (sbits[j][t]).
__global__ __launch_bounds__(256) void k_hidden_step(BpttArgs a, uint32_t t, const float *vprev,
                                                     const float *sprev, float *v_out, float *s_out) {
  const uint32_t j = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // wave-uniform
  if (j >= a.H) return;
  const uint32_t b = lane_id();
  const bool binary = a.smooth == 0;
  float acc = a.iin[((size_t)t * a.H + j) * 64 + b];
  if (sprev) {
    if (binary)
      acc = ordered_mask_sum(acc, a.rec_t_ptr[j], a.rec_t_ptr[j + 1], a.rec_t_src, a.w_rec_t, a.sbits, a.T, t - 1);
    else
      acc = ordered_gather_pipe(acc, a.rec_t_ptr[j], a.rec_t_ptr[j + 1], a.rec_t_src, a.w_rec_t, sprev, b);
  }
  const float vp = vprev ? vprev[(size_t)j * 64 + b] : 0.0f;
  const float sp = sprev ? sprev[(size_t)j * 64 + b] : 0.0f;
  float v = a.beta * vp;
  v = v + acc;
  v = v - a.theta * sp;
  v_out[(size_t)j * 64 + b] = v;
  if (s_out) {
    const float sv = spike_fn(v - a.theta, a.slope, a.smooth != 0);
    s_out[(size_t)j * 64 + b] = sv;
    if (binary) {
      const uint64_t m = __ballot(b < a.B && sv != 0.0f);
      if (b == 0) a.sbits[(size_t)j * a.T + t] = m;
    }
  }
}

// The hidden step in spiking mode with the ELL copy of the recurrent in-edges: the row of
// neuron j sits at j * ell_w, so its sources and weights are requested at once, together
// with iin, the state and the previous step's masks of all H neurons, which the workgroup
// stages in LDS (one memory round trip in all, where the CSR form needs the row bounds,
// then the edges, then the masks).  Each lane then reads its edge's mask from LDS, and the
// terms are added in row order, one add and one select each, as in ordered_mask_sum.
// kChunks = ell_w / 64.  The step writes its masks in both layouts.
template <int kChunks>
__global__ __launch_bounds__(256) void k_hidden_step_ell(BpttArgs a, uint32_t t, const float *vprev,
                                                         const float *sprev, float *v_out, float *s_out) {
  extern __shared__ uint64_t prev_masks[];  // [H]: step t - 1
  const uint32_t j = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // wave-uniform
  // every wave reaches the barrier; one past the last neuron loads neuron 0's data and
  // stores nothing
  const bool live = j < a.H;
  const uint32_t jl = live ? j : 0u;
  const uint32_t b = lane_id();
  const size_t jb = (size_t)jl * 64 + b;
  float acc = a.iin[(size_t)t * a.H * 64 + jb];
  const float vp = vprev ? vprev[jb] : 0.0f;
  const float sp = sprev ? sprev[jb] : 0.0f;
  int32_t src[kChunks];
  float wt[kChunks];
#pragma unroll
  for (int c = 0; c < kChunks; ++c) {
    const size_t x = (size_t)jl * a.ell_w + (uint32_t)c * kWave + b;
    src[c] = a.ell_src[x];
    wt[c] = a.ell_wt[x];
  }
  const uint32_t len = a.ell_len[jl];
  if (sprev) {
    // four loads per thread in flight, from indices clamped into the row
    const uint64_t *row = a.sbits_t + (size_t)(t - 1) * a.H;
    for (uint32_t base = 0; base < a.H; base += 4u * 256u) {
      uint64_t v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = row[std::min<uint32_t>(base + (uint32_t)q * 256u + threadIdx.x, a.H - 1)];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t i = base + (uint32_t)q * 256u + threadIdx.x;
        if (i < a.H) prev_masks[i] = v[q];
      }
    }
  }
  __syncthreads();
  if (sprev && live) {
    uint64_t m[kChunks];
#pragma unroll
    for (int c = 0; c < kChunks; ++c) m[c] = (uint32_t)c * kWave + b < len ? prev_masks[src[c]] : 0u;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const uint32_t n = len > (uint32_t)c * kWave ? std::min<uint32_t>(len - (uint32_t)c * kWave, kWave) : 0u;
#pragma unroll 8
      for (uint32_t u = 0; u < ((n + 7u) & ~7u); ++u) {
        const float sum = acc + __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wt[c]), (int)u));
        acc = __builtin_amdgcn_inverse_ballot_w64(lane_read64(m[c], u)) ? sum : acc;
      }
    }
  }
  if (!live) return;
  float v = a.beta * vp;
  v = v + acc;
  v = v - a.theta * sp;
  v_out[jb] = v;
  if (s_out) {
    const float sv = spike_fn(v - a.theta, a.slope, false);
    s_out[jb] = sv;
    const uint64_t mk = __ballot(b < a.B && sv != 0.0f);
    if (b == 0) {
      a.sbits[(size_t)j * a.T + t] = mk;
      a.sbits_t[(size_t)t * a.H + j] = mk;
    }
  }
}

// ---- the event-driven forward pass ------------------------------------------------------
// In spiking mode with at most kEventMaxNeurons hidden neurons the forward pass works on what
// is not zero.  Batch elements do not interact in it, so a workgroup steps one of them through
// the whole sequence, with nothing to wait for outside itself.  Weights are held as dense
// rows (Hp columns, zeros off the synapses): a presynaptic spike adds its row to the
// currents of all neurons, one neuron per lane, sources in ascending order, which is the
// defined sum (a term off the synapses adds +0 to a sum that starts from +0, and w * 1 = w).
//   vall  [T][B][Hp]  the input current of every step, replaced by the membrane potential
//   spk   [B][T][nw]  spikes of every step, 64 neurons per word

__device__ __forceinline__ size_t row_index(const BpttArgs &a, uint32_t t, uint32_t b) {
  return ((size_t)t * a.B + b) * a.Hp;
}

// The caller's weights into the plan's layouts, edge e at pos[e]: dense rows of the input and
// recurrent weights, and the target-major pairs of the many-spikes form.
__global__ void k_scatter_weights(BpttArgs a) {
  const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  // k_transpose_x sets flags[0] for inputs other than 0 and 1, flags[2] for readout weights that
  // are not finite
  if (e < 3) a.flags[e] = 0;
  if (e < a.nnz_in) a.dense_in[a.in_pos[e]] = a.w_in[e];
  if (e < a.nnz_rec) {
    const float w = a.w_rec[e];
    a.dense_rec[a.rec_pos[e]] = w;
    a.col_pair[a.col_pos[e]].y = __float_as_uint(w);
  }
}

// Input-projection current of every (batch element, step) from binary inputs: a wavefront
// finds the active inputs of 64 at a time by a ballot and adds their dense rows, 16 bytes per
// lane and block of 256 columns, up to four rows and kInputBlocks blocks in flight.  Bound:
// the rows' way from L2 (280,000 active inputs x 4 KB at 64 x 250 x 700 -> 1,024).
constexpr int kInputBlocks = 4;
__global__ __launch_bounds__(256) void k_input_rows(BpttArgs a, const float *x) {
  if (a.flags[0] != 0) return;  // not binary: k_input_current_values
  const uint32_t bt = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (bt >= a.B * a.T) return;
  const uint32_t lane = lane_id();
  const uint32_t nb = std::min<uint32_t>(kInputBlocks, a.Hp / 256 - blockIdx.y * kInputBlocks);
  const size_t col = (size_t)blockIdx.y * kInputBlocks * 256 + lane * 4;
  const float *xr = x + (size_t)bt * a.C;
  float4 acc[kInputBlocks];
#pragma unroll
  for (int q = 0; q < kInputBlocks; ++q) acc[q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  float xv = lane < a.C ? xr[lane] : 0.0f;
  for (uint32_t c0 = 0; c0 < a.C; c0 += kWave) {
    uint64_t m = __ballot(xv != 0.0f);
    xv = c0 + kWave + lane < a.C ? xr[c0 + kWave + lane] : 0.0f;  // the next 64
    while (m) {
      const uint32_t n = std::min<uint32_t>(4u, (uint32_t)__popcll(m));  // uniform
      float4 w[4][kInputBlocks];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if ((uint32_t)u < n) {
          const float *row = a.dense_in + (size_t)(c0 + (uint32_t)__builtin_ctzll(m)) * a.Hp + col;
          m &= m - 1;
#pragma unroll
          for (int q = 0; q < kInputBlocks; ++q)
            if ((uint32_t)q < nb) w[u][q] = *reinterpret_cast<const float4 *>(row + q * 256);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if ((uint32_t)u < n) {
#pragma unroll
          for (int q = 0; q < kInputBlocks; ++q) {
            if ((uint32_t)q < nb) {
              acc[q].x = acc[q].x + w[u][q].x;
              acc[q].y = acc[q].y + w[u][q].y;
              acc[q].z = acc[q].z + w[u][q].z;
              acc[q].w = acc[q].w + w[u][q].w;
            }
          }
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kInputBlocks; ++q)
    if ((uint32_t)q < nb) *reinterpret_cast<float4 *>(a.vall + row_index(a, bt % a.T, bt / a.T) + col + q * 256) = acc[q];
}

// All hidden steps of one batch element: one workgroup, a wavefront per kPer words of 64
// neurons (neuron 64 q + lane of its range), one barrier per step, at which the step's spikes
// are published as words in LDS.  Every wavefront takes the sources off the words by itself,
// mostly with scalar instructions, so few wavefronts with several words each do better than
// one per word (1,024 neurons: 1.29 us per step with 8 wavefronts, 1.35 with 4, 1.6 with 16).  Global memory other
// than weight rows is touched once per kSeqChunk steps: the chunk's input currents, requested
// a chunk ahead, pass through LDS (so that a step can index them), where the membranes replace
// them until the chunk is written out with its spike words; a store in every step would be
// waited for by the step's row reads.  Per step a wavefront reads the previous step's words,
// takes its sources off them in ascending order and adds their rows, up to kSeqRows in
// flight; with more sources than twice the longest column it walks the columns (target-major
// pairs) and tests each source's bit instead.  64 x 250 x 1,024 with 3.7 spikes per step: 323
// us, where a launch per step took 1,540; 19 x 103 x 201: 49 us (370).
constexpr uint32_t kSeqChunk = 16;
constexpr uint32_t kSeqThreads = kEventMaxNeurons / 4;
constexpr int kSeqRows = 4;
template <int kPer>
__global__ __launch_bounds__(kSeqThreads) void k_hidden_seq(BpttArgs a) {
  extern __shared__ float cur_s[];  // [kSeqChunk][Hp]
  __shared__ uint64_t words_s[2 * kSeqChunk][kEventMaxNeurons / 64];  // step mod 2 chunks
  const uint32_t b = blockIdx.x, tid = threadIdx.x, lane = lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const size_t step_rows = (size_t)a.B * a.Hp;
  float *vrow = a.vall + row_index(a, 0, b);
  uint64_t *srow = a.spk + (size_t)b * a.T * a.nw;
  float v[kPer], sp[kPer], ahead[kSeqChunk][kPer];
  const uint32_t w0 = wave * kPer;            // this wavefront's words [w0, w0 + kPer)
  const uint32_t col0 = w0 * kWave + lane;    // its neurons col0 + 64 q (inside Hp: whole
                                              // wavefronts of words, kPer of them divide Hp)
#pragma unroll
  for (int q = 0; q < kPer; ++q) v[q] = sp[q] = 0.0f;
  auto request = [&](uint32_t t0) {
#pragma unroll
    for (uint32_t k = 0; k < kSeqChunk; ++k)
#pragma unroll
      for (int q = 0; q < kPer; ++q) ahead[k][q] = vrow[std::min<uint32_t>(t0 + k, a.T - 1) * step_rows + col0 + (uint32_t)q * kWave];
  };
  // membranes and spike words of the steps [t0, t1), t0 a chunk's first step, after a barrier
  auto flush = [&](uint32_t t0, uint32_t t1) {
#pragma unroll
    for (uint32_t k = 0; k < kSeqChunk; ++k)
#pragma unroll
      for (int q = 0; q < kPer; ++q)
        if (t0 + k < t1) vrow[(t0 + k) * step_rows + col0 + (uint32_t)q * kWave] = cur_s[k * a.Hp + col0 + (uint32_t)q * kWave];
    for (uint32_t x = tid; x < (t1 - t0) * a.nw; x += blockDim.x)
      srow[(size_t)t0 * a.nw + x] = words_s[(t0 + x / a.nw) % (2 * kSeqChunk)][x % a.nw];
  };
  request(0);
  for (uint32_t t = 0; t < a.T; ++t) {
    const uint32_t k = t % kSeqChunk;
    if (k == 0) {  // a lane reads back only what it wrote
      if (t) flush(t - kSeqChunk, t);
#pragma unroll
      for (uint32_t u = 0; u < kSeqChunk; ++u)
#pragma unroll
        for (int q = 0; q < kPer; ++q)
          cur_s[u * a.Hp + col0 + (uint32_t)q * kWave] = ahead[u][q];
      if (t + kSeqChunk < a.T) request(t + kSeqChunk);
    }
    float acc[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) acc[q] = cur_s[k * a.Hp + col0 + (uint32_t)q * kWave];
    if (t) {
      const uint64_t *prev = words_s[(t - 1) % (2 * kSeqChunk)];
      const uint64_t mine = lane < a.nw ? prev[lane] : 0ull;
      uint64_t any = __ballot(mine != 0);  // words with spikes
      bool columns = false;
      if ((uint32_t)__popcll(any) * 64u > 2u * a.col_w) {  // the count can exceed the limit
        const uint32_t incl = wave_inclusive_scan((uint32_t)__popcll(mine));
        columns = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1) > 2u * a.col_w;
      }
      if (columns) {
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
          const uint2 *pairs = a.col_pair + col0 + (uint32_t)q * kWave;
#pragma unroll 4
          for (uint32_t r = 0; r < a.col_w; ++r) {
            const uint2 e = pairs[(size_t)r * a.Hp];  // padding: source 0, weight 0
            const float sum = acc[q] + __uint_as_float(e.y);
            acc[q] = (prev[e.x >> 6] >> (e.x & 63u)) & 1u ? sum : acc[q];
          }
        }
      } else {
        uint64_t word = 0;
        uint32_t at = 0;
        while (any) {
          float w[kSeqRows][kPer];
          uint32_t n = 0;
#pragma unroll
          for (int u = 0; u < kSeqRows; ++u) {
            if (any) {  // uniform
              if (!word) {
                at = (uint32_t)__builtin_ctzll(any);
                word = lane_read64(mine, at);
              }
              const uint32_t src = at * 64u + (uint32_t)__builtin_ctzll(word);
              word &= word - 1;
              if (!word) any &= any - 1;
              const float *row = a.dense_rec + (size_t)src * a.Hp;
#pragma unroll
              for (int q = 0; q < kPer; ++q) w[u][q] = row[col0 + (uint32_t)q * kWave];
              n = (uint32_t)u + 1u;
            }
          }
#pragma unroll
          for (int u = 0; u < kSeqRows; ++u)
            if ((uint32_t)u < n) {
#pragma unroll
              for (int q = 0; q < kPer; ++q) acc[q] = acc[q] + w[u][q];
            }
        }
      }
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const uint32_t j = col0 + (uint32_t)q * kWave;
      float vn = a.beta * v[q];
      vn = vn + acc[q];
      vn = vn - a.theta * sp[q];
      v[q] = vn;
      const bool spike = j < a.H && spike_fn(vn - a.theta, a.slope, false) != 0.0f;
      sp[q] = spike ? 1.0f : 0.0f;
      const uint64_t m = __ballot(spike);
      if (lane == 0) words_s[t % (2 * kSeqChunk)][w0 + (uint32_t)q] = m;
      cur_s[k * a.Hp + j] = vn;
    }
    __syncthreads();
  }
  flush((a.T - 1) / kSeqChunk * kSeqChunk, a.T);
}

// The busy form of the hidden steps, one launch each: lanes are batch elements and a wavefront one
// neuron, so that the step costs by neurons and synapses, whatever the activity, on all compute
// units (k_hidden_step_ell with other arrays).  Input currents and membranes are held in the slices
// of the backward pass's sg and lamv, which are free until then; spikes are batch masks,
// sbits_t[t][j]; k_busy_rows takes both to the rows of the event-driven form when all steps are
// done.  (In vall itself, where a neuron's lanes lie Hp floats apart, a step of 700 neurons took
// 0.4 us longer.)  kChunks = ell_w / 64, or 0 for rows that only the CSR form holds.  6.2 us per step
// of 1,024 neurons with rows of 102, at any activity; k_hidden_seq takes 1.3 us at 4 spikes a step,
// 6.5 at 43 and 32 at 268.
template <int kChunks>
__global__ __launch_bounds__(256) void k_hidden_step_busy(BpttArgs a, uint32_t t) {
  extern __shared__ uint64_t prev_masks[];  // [H]: step t - 1
  const uint32_t j = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // wave-uniform
  const bool live = j < a.H;
  const uint32_t jl = live ? j : 0u;
  const uint32_t b = lane_id();
  const size_t own = slice_index(a, t, std::min<uint32_t>(b, a.B - 1u), jl);
  float acc = a.sg[own];
  const float vp = t ? a.lamv[own - (size_t)a.S * a.H * 8] : 0.0f;
  int32_t src[kChunks ? kChunks : 1];
  float wt[kChunks ? kChunks : 1];
  uint32_t len = 0;
  if (kChunks) {
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const size_t x = (size_t)jl * a.ell_w + (uint32_t)c * kWave + b;
      src[c] = a.ell_src[x];
      wt[c] = a.ell_wt[x];
    }
    len = a.ell_len[jl];
  }
  const uint64_t *row = a.sbits_t + (size_t)(t ? t - 1 : 0) * a.H;
  if (t) {
    for (uint32_t base = 0; base < a.H; base += 4u * 256u) {
      uint64_t v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = row[std::min<uint32_t>(base + (uint32_t)q * 256u + threadIdx.x, a.H - 1)];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t i = base + (uint32_t)q * 256u + threadIdx.x;
        if (i < a.H) prev_masks[i] = v[q];
      }
    }
  }
  __syncthreads();
  if (!live) return;
  float sp = 0.0f;
  if (t) {
    sp = (prev_masks[jl] >> b) & 1u ? 1.0f : 0.0f;
    if (kChunks) {
      uint64_t m[kChunks ? kChunks : 1];
#pragma unroll
      for (int c = 0; c < kChunks; ++c) m[c] = (uint32_t)c * kWave + b < len ? prev_masks[src[c]] : 0u;
#pragma unroll
      for (int c = 0; c < kChunks; ++c) {
        const uint32_t n = len > (uint32_t)c * kWave ? std::min<uint32_t>(len - (uint32_t)c * kWave, kWave) : 0u;
#pragma unroll 8
        for (uint32_t u = 0; u < ((n + 7u) & ~7u); ++u) {
          const float sum = acc + __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wt[c]), (int)u));
          acc = __builtin_amdgcn_inverse_ballot_w64(lane_read64(m[c], u)) ? sum : acc;
        }
      }
    } else {
      acc = ordered_mask_sum(acc, a.rec_t_ptr[j], a.rec_t_ptr[j + 1], a.rec_t_src, a.w_rec_t, row, 1, 0);
    }
  }
  float v = a.beta * vp;
  v = v + acc;
  v = v - a.theta * sp;
  if (b < a.B) a.lamv[own] = v;
  const uint64_t mk = __ballot(b < a.B && spike_fn(v - a.theta, a.slope, false) != 0.0f);
  if (b == 0) a.sbits_t[(size_t)t * a.H + j] = mk;
}

// The busy form's membranes and spikes as rows and words of every batch element: a workgroup per
// (word of 64 neurons, step) transposes the step's slices through LDS.
__global__ __launch_bounds__(256) void k_busy_rows(BpttArgs a) {
  __shared__ float tile[64][65];  // [b][neuron]
  const uint32_t w = blockIdx.x, t = blockIdx.y, n = std::min<uint32_t>(64u, a.H - w * 64u);
  for (uint32_t x = threadIdx.x; x < a.S * 512u; x += 256u) {
    const uint32_t j = (x & 511u) >> 3, b = (x >> 9) * 8u + (x & 7u);
    if (j < n) tile[b][j] = a.lamv[slice_index(a, t, b, w * 64u + j)];
  }
  __syncthreads();
  const uint32_t lane = lane_id();
  for (uint32_t b = threadIdx.x / kWave; b < a.B; b += 4u) {
    const float v = lane < n ? tile[b][lane] : 0.0f;
    const uint64_t word = __ballot(lane < n && spike_fn(v - a.theta, a.slope, false) != 0.0f);
    if (lane < n) a.vall[row_index(a, t, b) + w * 64u + lane] = v;
    if (lane == 0) a.spk[((size_t)b * a.T + t) * a.nw + w] = word;
  }
}

// Batch masks of the hidden spikes from the words of every batch element: a workgroup per
// (word, kMaskBlock steps) sets the few spikes' bits in LDS and writes the 64 neurons' masks
// of its steps, contiguous per neuron.
constexpr uint32_t kMaskBlock = 16;
__global__ __launch_bounds__(256) void k_spike_masks(BpttArgs a) {
  __shared__ unsigned long long mask[64][kMaskBlock];
  const uint32_t w = blockIdx.x, t0 = blockIdx.y * kMaskBlock, tid = threadIdx.x;
  const uint32_t tl = tid % kMaskBlock, t = t0 + tl;
  if (w == 0 && t0 == 0 && tid == 0) a.flags[3] = 0;  // k_lam_u sets it for adjoints that are not finite
  uint64_t word[64 * kMaskBlock / 256];  // (step tl, batch elements tid / 16 + 16 q)
#pragma unroll
  for (uint32_t q = 0; q < 64 * kMaskBlock / 256; ++q) {
    const uint32_t b = tid / kMaskBlock + q * (256 / kMaskBlock);
    word[q] = b < a.B && t < a.T ? a.spk[((size_t)b * a.T + t) * a.nw + w] : 0ull;
  }
  for (uint32_t x = tid; x < 64 * kMaskBlock; x += 256) (&mask[0][0])[x] = 0ull;
  __syncthreads();
#pragma unroll
  for (uint32_t q = 0; q < 64 * kMaskBlock / 256; ++q)
    for (uint64_t m = word[q]; m; m &= m - 1)
      atomicOr(&mask[__builtin_ctzll(m)][tl], 1ull << (tid / kMaskBlock + q * (256 / kMaskBlock)));
  __syncthreads();
  for (uint32_t x = tid; x < 64 * kMaskBlock; x += 256) {
    const uint32_t i = w * 64u + x / kMaskBlock;
    if (i < a.H && t0 + x % kMaskBlock < a.T) a.sbits[(size_t)i * a.T + t0 + x % kMaskBlock] = (&mask[0][0])[x];
  }
}

// Readout drive of every (batch element, step) from its spikes: ro[b][t][o] = sum of the
// spiking neurons' readout weights, ascending; a wavefront per (b, t), lanes = readouts.  That is
// the defined sum of s w over all neurons while the weights are finite; with one that is not,
// every term is formed (0 w is then no zero).
__global__ __launch_bounds__(256) void k_readout_events(BpttArgs a, float *ro) {
  const uint32_t bt = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (bt >= a.B * a.T) return;
  const uint32_t lane = lane_id();
  const uint64_t mine = lane < a.nw ? a.spk[(size_t)bt * a.nw + lane] : 0ull;
  const bool every = a.flags[2] != 0;
  for (uint32_t o0 = 0; o0 < a.O; o0 += kWave) {
    const uint32_t o = std::min<uint32_t>(o0 + lane, a.O - 1);
    float acc = 0.0f;
    uint64_t any = __ballot(mine != 0), word = 0;
    uint32_t at = 0;
    while (any) {
      float w[4];
      uint32_t n = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (any) {
          if (!word) {
            at = (uint32_t)__builtin_ctzll(any);
            word = lane_read64(mine, at);
          }
          w[u] = a.w_out[(size_t)(at * 64u + (uint32_t)__builtin_ctzll(word)) * a.O + o];
          word &= word - 1;
          if (!word) any &= any - 1;
          n = (uint32_t)u + 1u;
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if ((uint32_t)u < n) acc = acc + w[u];
    }
    if (every) {
      acc = 0.0f;
      for (uint32_t i = 0; i < a.H; ++i) {
        const float on = (lane_read64(mine, i >> 6) >> (i & 63u)) & 1u ? 1.0f : 0.0f;
        acc = acc + on * a.w_out[(size_t)i * a.O + o];
      }
    }
    if (o0 + lane < a.O) ro[(size_t)bt * a.O + o0 + lane] = acc;
  }
}

// Readout drive of the busy form, from its masks: lanes are batch elements, a wavefront takes
// kMaskOuts readouts of a step over all neurons, ascending, with one add and one select each.  The
// masks and weights of 64 neurons arrive one per lane and reach the wavefront by lane reads, as in
// ordered_mask_sum; the next 64 are requested ahead.  80 us for 64 x 250 steps, 1,024 neurons and 20
// readouts, whatever the spikes; k_readout_events, which reads a row of weights per spike, takes 8 us
// at 4 spikes a step and 235 at 408.
constexpr int kMaskOuts = 4;
__global__ __launch_bounds__(64) void k_readout_masks(BpttArgs a, float *ro) {
  const uint32_t t = blockIdx.x, o0 = blockIdx.y * kMaskOuts, b = threadIdx.x;
  const uint64_t *masks = a.sbits_t + (size_t)t * a.H;
  const uint32_t last = std::min<uint32_t>(kMaskOuts, a.O - o0) - 1u;
  const bool every = a.flags[2] != 0;  // as k_readout_events
  float acc[kMaskOuts] = {}, w[kMaskOuts], wn[kMaskOuts];
  uint64_t m, mn;
  auto request = [&](uint32_t base) {  // past the last neuron: an empty mask, a weight of 0
    const uint32_t i = base + b;
    mn = i < a.H ? masks[i] : 0ull;
#pragma unroll
    for (uint32_t q = 0; q < kMaskOuts; ++q)
      wn[q] = i < a.H ? a.w_out[(size_t)i * a.O + o0 + std::min(q, last)] : 0.0f;
  };
  request(0);
  for (uint32_t base = 0; base < a.H; base += kWave) {
    m = mn;
#pragma unroll
    for (int q = 0; q < kMaskOuts; ++q) w[q] = wn[q];
    if (base + kWave < a.H) request(base + kWave);
    if (every) {
      for (uint32_t u = 0; u < kWave; ++u) {
        const float on = __builtin_amdgcn_inverse_ballot_w64(lane_read64(m, u)) ? 1.0f : 0.0f;
#pragma unroll
        for (int q = 0; q < kMaskOuts; ++q)
          acc[q] = acc[q] + on * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w[q]), (int)u));
      }
    } else {
#pragma unroll 8
      for (uint32_t u = 0; u < kWave; ++u) {
        const bool on = __builtin_amdgcn_inverse_ballot_w64(lane_read64(m, u));
#pragma unroll
        for (int q = 0; q < kMaskOuts; ++q) {
          const float sum = acc[q] + __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w[q]), (int)u));
          acc[q] = on ? sum : acc[q];
        }
      }
    }
  }
  if (b < a.B)
    for (uint32_t q = 0; q <= last; ++q) ro[((size_t)b * a.T + t) * a.O + o0 + q] = acc[q];
}

// Set bits of kActSamples words of an array of n, by a wavefront: eight words at each of a number
// of scattered places, as a compute unit has some 64 line reads in flight, and in few
// instructions, which all come from memory (in two kilobytes of them the sample took longer than
// the scan of a short pass).
__device__ __forceinline__ uint32_t sample_bits(const uint64_t *words, uint64_t n) {
  constexpr uint32_t kEach = kActSamples / kWave;
  const uint32_t most = (uint32_t)std::min<uint64_t>(n, 8), places = (uint32_t)std::min<uint64_t>(n, UINT32_MAX) - most + 1;
  const uint64_t *own = words + std::min<uint32_t>(lane_id() & 7u, most - 1);
  uint64_t w[kEach];
#pragma unroll
  for (uint32_t k = 0; k < kEach; ++k) w[k] = own[__umulhi((k * 8u + (lane_id() >> 3)) * 0x9E3779B9u, places)];
  uint32_t count = 0;
#pragma unroll
  for (uint32_t k = 0; k < kEach; ++k) count += (uint32_t)__popcll(w[k]);
  return wave_sum(count);
}

// The leaky readout's scan (as k_readout_scan) over ro[b][t][o]: block (2 + b, 64 readouts).  Beside
// it two blocks take the pass's activity, a sample of the inputs and of the hidden spikes, to host
// memory: what the next pass's way is chosen by.
__global__ __launch_bounds__(64) void k_readout_scan_events(BpttArgs a, const float *ro) {
  if (blockIdx.x < 2) {  // (first, so that the other blocks branch without waiting for an argument)
    if (blockIdx.y) return;
    const bool in = blockIdx.x == 0;
    const uint32_t bits = sample_bits(in ? a.xbits : a.spk, in ? (uint64_t)a.C * a.T : (uint64_t)a.B * a.T * a.nw);
    if (threadIdx.x == 0) {
      a.act_out[blockIdx.x] = bits;
      if (blockIdx.x == 0) a.act_out[2] = a.flags[0];
    }
    return;
  }
  const uint32_t b = blockIdx.x - 2, o = blockIdx.y * 64u + threadIdx.x;
  const float *r0 = ro + (size_t)b * a.T * a.O + std::min<uint32_t>(o, a.O - 1);
  float u = 0.0f, m = 0.0f;
  uint32_t tm = 0;
  auto step = [&](uint32_t t, float r) {
    float ut = a.beta_out * u;
    ut = ut + r;
    u = ut;
    if (t == 0 || ut > m) {
      m = ut;
      tm = t;
    }
  };
  constexpr uint32_t kAhead = 16;  // drives requested before the steps that use them
  float r[kAhead], nx[kAhead];
#pragma unroll
  for (uint32_t q = 0; q < kAhead; ++q) r[q] = r0[(size_t)std::min<uint32_t>(q, a.T - 1) * a.O];
  for (uint32_t t = 0; t < a.T; t += kAhead) {
#pragma unroll
    for (uint32_t q = 0; q < kAhead; ++q) nx[q] = r0[(size_t)std::min<uint32_t>(t + kAhead + q, a.T - 1) * a.O];
#pragma unroll
    for (uint32_t q = 0; q < kAhead; ++q)
      if (t + q < a.T) step(t + q, r[q]);
#pragma unroll
    for (uint32_t q = 0; q < kAhead; ++q) r[q] = nx[q];
  }
  if (o < a.O) {
    a.m[(size_t)b * a.O + o] = m;
    a.tmax[(size_t)b * a.O + o] = (int32_t)tm;
  }
}

// Membrane checkpoints [segment][H][64] of the latest forward pass, for the trace.
__global__ void k_trace_v(BpttArgs a) {
  const uint64_t x = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t n_seg = (a.T + a.K - 1) / a.K;
  if (x >= (uint64_t)n_seg * a.H * 64) return;
  const uint32_t b = (uint32_t)(x & 63u), j = (uint32_t)((x >> 6) % a.H), seg = (uint32_t)((x >> 6) / a.H);
  const uint32_t t = std::min<uint32_t>((seg + 1) * a.K - 1, a.T - 1);
  a.vck[x] = b < a.B ? a.vall[row_index(a, t, b) + j] : 0.0f;
}

// Backward recomputation of one checkpoint segment [t0, t0 + len).  The spikes of every
// step are stored, so the currents of all the segment's steps are independent: these
// kernels compute them in parallel, each exactly as k_hidden_step does (input part, then
// the recurrent in-edges over s_{t-1} in ascending source order), into cur[k][j][b].  In
// spiking mode k_seg_current takes the terms from the spike masks the forward pass
// wrote, a wavefront per (block of kMaskSteps steps, j); in smooth mode
// k_seg_current_values gathers the values, a wavefront per (k, j).
__global__ __launch_bounds__(256) void k_seg_current(BpttArgs a, uint32_t t0, uint32_t len, float *cur) {
  const uint64_t w = (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t n_blocks = (len + kMaskSteps - 1) / kMaskSteps;
  if (w >= (uint64_t)n_blocks * a.H) return;
  const uint32_t k0 = (uint32_t)(w / a.H) * kMaskSteps, j = (uint32_t)(w % a.H);
  const uint32_t nt = std::min<uint32_t>(kMaskSteps, len - k0);
  const uint32_t b = lane_id();
  float acc[kMaskSteps];
#pragma unroll
  for (int u = 0; u < kMaskSteps; ++u)
    acc[u] = (uint32_t)u < nt ? a.iin[((size_t)(t0 + k0 + u) * a.H + j) * 64 + b] : 0.0f;
  const float first = acc[0];
  // column t - 1 of step t; at t = 0 the masks read (entries before the array's start
  // for j = 0) are not used: that step has no recurrent term
  ordered_mask_sum_steps(acc, a.rec_t_ptr[j], a.rec_t_ptr[j + 1], a.rec_t_src, a.w_rec_t, a.sbits, a.T,
                         (int64_t)(t0 + k0) - 1);
  if (t0 + k0 == 0) acc[0] = first;
#pragma unroll
  for (int u = 0; u < kMaskSteps; ++u)
    if ((uint32_t)u < nt) cur[((size_t)(k0 + u) * a.H + j) * 64 + b] = acc[u];
}

__global__ __launch_bounds__(256) void k_seg_current_values(BpttArgs a, uint32_t t0, uint32_t len, float *cur) {
  const uint64_t w = (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (w >= (uint64_t)len * a.H) return;
  const uint32_t k = (uint32_t)(w / a.H), j = (uint32_t)(w % a.H), t = t0 + k;
  const uint32_t b = lane_id();
  float acc = a.iin[((size_t)t * a.H + j) * 64 + b];
  if (t > 0)
    acc = ordered_gather_sum(acc, a.rec_t_ptr[j], a.rec_t_ptr[j + 1], a.rec_t_src, a.w_rec_t,
                             a.s + (size_t)(t - 1) * a.H * 64, b);
  cur[w * 64 + b] = acc;
}

// ... then the membranes of the segment from the checkpoint before it (vprev; nullptr at
// step 0), one lane per (j, b), with k_hidden_step's operations in its order; vseg[k]
// holds the current of step t0 + k on entry and V_{t0+k} on return.
__global__ void k_seg_scan(BpttArgs a, uint32_t t0, uint32_t len, const float *vprev, float *vseg) {
  const uint32_t x = blockIdx.x * blockDim.x + threadIdx.x;  // j * 64 + b
  if (x >= a.H * 64) return;
  float v = vprev ? vprev[x] : 0.0f;
  for (uint32_t k = 0; k < len; ++k) {
    const uint32_t t = t0 + k;
    const float sp = t ? a.s[(size_t)(t - 1) * a.H * 64 + x] : 0.0f;
    float vn = a.beta * v;
    vn = vn + vseg[(size_t)k * a.H * 64 + x];
    vn = vn - a.theta * sp;
    vseg[(size_t)k * a.H * 64 + x] = vn;
    v = vn;
  }
}

// Readout drive of every step: ro[t][o][b] = sum_i s[t][i][b] w_out[i][o], ascending i;
// the loads of 16 consecutive i are issued before their terms are added in order.
__global__ void k_readout_drive(BpttArgs a, float *ro) {
  const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (uint64_t)a.T * a.O * 64) return;
  const uint32_t b = (uint32_t)(idx & 63u);
  const uint64_t to = idx >> 6;
  const uint32_t o = (uint32_t)(to % a.O), t = (uint32_t)(to / a.O);
  const float *st = a.s + (size_t)t * a.H * 64 + b;
  const float *wo = a.w_out + o;
  float acc = 0.0f;
  uint32_t i = 0;
  for (; i + 16 <= a.H; i += 16) {
    float sv[16], wv[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      sv[u] = st[(size_t)(i + u) * 64];
      wv[u] = wo[(size_t)(i + u) * a.O];
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) acc = acc + sv[u] * wv[u];
  }
  for (; i < a.H; ++i) acc = acc + st[(size_t)i * 64] * wo[(size_t)i * a.O];
  ro[idx] = acc;
}

// Leaky readout and its maximum over time (first step attaining it): block o, lane b.
__global__ void k_readout_scan(BpttArgs a, const float *ro) {
  const uint32_t o = blockIdx.x, b = threadIdx.x;
  if (b >= a.B) return;
  float u = 0.0f, m = 0.0f;
  uint32_t tm = 0;
  auto step = [&](uint32_t t, float r) {
    float ut = a.beta_out * u;
    ut = ut + r;
    u = ut;
    if (t == 0 || ut > m) {
      m = ut;
      tm = t;
    }
  };
  uint32_t t = 0;
  for (; t + 8 <= a.T; t += 8) {  // eight drives requested before the eight steps
    float r[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) r[q] = ro[((size_t)(t + q) * a.O + o) * 64 + b];
#pragma unroll
    for (int q = 0; q < 8; ++q) step(t + q, r[q]);
  }
  for (; t < a.T; ++t) step(t, ro[((size_t)t * a.O + o) * 64 + b]);
  a.m[(size_t)b * a.O + o] = m;
  a.tmax[(size_t)b * a.O + o] = (int32_t)tm;
}

// Softmax cross entropy of the maxima, its gradient dL/dmax = (p - onehot) / B, and the
// mean loss; one block of 64 threads (lane b).
__global__ void k_loss(BpttArgs a, const int32_t *labels, float *loss) {
  __shared__ float s_lb[64];
  const uint32_t b = threadIdx.x;
  if (b < a.B) {
    const float *m = a.m + (size_t)b * a.O;
    float mx = m[0];
    for (uint32_t k = 1; k < a.O; ++k) mx = fmaxf(mx, m[k]);
    float z = 0.0f;
    for (uint32_t k = 0; k < a.O; ++k) z += expf(m[k] - mx);
    const int32_t y = labels[b];
    const bool valid = y >= 0 && (uint32_t)y < a.O;  // an invalid label yields NaN
    s_lb[b] = valid ? mx + logf(z) - m[y] : __int_as_float(0x7fc00000);
    for (uint32_t k = 0; k < a.O; ++k) {
      const float p = expf(m[k] - mx) / z;
      a.dm[(size_t)b * a.O + k] = valid ? (p - ((int32_t)k == y ? 1.0f : 0.0f)) / (float)a.B
                                        : __int_as_float(0x7fc00000);
    }
  }
  __syncthreads();
  if (b == 0) {
    float sum = 0.0f;
    for (uint32_t k = 0; k < a.B; ++k) sum += s_lb[k];
    *loss = sum / (float)a.B;
  }
}

// Readout adjoint: lamu[t][o][b] = g_t + beta_out lamu[t+1], g_t = dm at the max step,
// scaled by the incoming gradient of the loss; block o, lane b (zeros for b >= B).
__global__ void k_lam_u(BpttArgs a, const float *g_loss) {
  const uint32_t o = blockIdx.x, b = threadIdx.x;
  const float scale = g_loss ? *g_loss : 1.0f;
  const float g = b < a.B ? a.dm[(size_t)b * a.O + o] * scale : 0.0f;
  const int32_t tm = b < a.B ? a.tmax[(size_t)b * a.O + o] : -1;
  float nxt = 0.0f;
  for (int32_t t = (int32_t)a.T - 1; t >= 0; --t) {
    nxt = (t == tm ? g : 0.0f) + a.beta_out * nxt;
    a.lamu[((size_t)t * a.O + o) * 64 + b] = nxt;
  }
  // (a value that is not finite makes every later one so)
  if (!finite_f32(nxt)) atomicOr(a.flags + 3, 1u);
}

// Readout part of the spike adjoint of every step, the first terms of the sum that
// k_adjoint_step completes: dsr[t][i][b] = sum_o w_out[i][o] lamu[t][o][b], ascending o
// from +0.  It does not depend on the membrane adjoint, so all steps run in parallel (a
// wavefront per (t, i)), ahead of the sequential adjoint steps.
__global__ __launch_bounds__(256) void k_readout_adjoint(BpttArgs a, float *dsr) {
  const uint64_t w = (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (w >= (uint64_t)a.T * a.H) return;
  const uint32_t t = (uint32_t)(w / a.H), i = (uint32_t)(w % a.H);
  const uint32_t b = lane_id();
  const float *lu = a.lamu + (size_t)t * a.O * 64 + b;
  // in ascending o, eight loads issued before their terms are added
  float ds = 0.0f;
  uint32_t o = 0;
  for (; o + 8 <= a.O; o += 8) {
    float wv[8], lv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      wv[u] = a.w_out[(size_t)i * a.O + o + u];
      lv[u] = lu[(size_t)(o + u) * 64];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) ds = ds + wv[u] * lv[u];
  }
  for (; o < a.O; ++o) ds = ds + a.w_out[(size_t)i * a.O + o] * lu[(size_t)o * 64];
  dsr[w * 64 + b] = ds;
}

// Membrane adjoint of step t: one wavefront per hidden neuron i, lane = batch.
// lam_next = lamV_{t+1} ([H][64], zeros for step T), v_t = V_t; lam_out = lamV_t holds
// the readout part of the spike adjoint (k_readout_adjoint) on entry and receives
// lamV_t.
__global__ __launch_bounds__(256) void k_adjoint_step(BpttArgs a, uint32_t t, const float *v_t,
                                                      const float *lam_next, float *lam_out) {
  const uint32_t i = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // wave-uniform
  if (i >= a.H) return;
  const uint32_t b = lane_id();
  float ds = lam_out[(size_t)i * 64 + b];  // the readout terms, in ascending o
  // the neuron's own values are requested before the gather, so that they are not a
  // round trip of their own after it (0.08 ms per iteration)
  const float ln = lam_next[(size_t)i * 64 + b];
  const float vt = v_t[(size_t)i * 64 + b];
  ds = ordered_gather_pipe(ds, a.rec_ptr[i], a.rec_ptr[i + 1], a.rec_col, a.w_rec, lam_next, b);
  if (!a.detach_reset) ds = ds - a.theta * ln;
  const float z = vt - a.theta;
  lam_out[(size_t)i * 64 + b] = a.beta * ln + surrogate(z, a.slope, a.smooth != 0) * ds;
}

// ---- the sliced membrane adjoint -------------------------------------------------------

// Readout part of the spike adjoint of every step (as k_readout_adjoint), in the sliced
// layout.  A workgroup per (block of 32 neurons, t): thread (neuron, b mod 8) keeps the sums
// of all slices; the readout adjoints of up to kReadoutChunk readouts and the block's
// weights are staged in LDS, the adjoints as [o][b mod 8][slice], so that a thread's slices
// of one readout are two 16-byte reads.  Bound: the store of the result (65 MB for 64 x 250
// x 1,024).
constexpr int kReadoutChunk = 32;
// In the event-driven form it also takes the surrogate derivative of its membranes, which
// come as rows of one batch element each, to the slices (an adjoint step that gathered them
// itself took 0.8 us longer).
__global__ __launch_bounds__(256) void k_readout_adjoint_slice(BpttArgs a, float *dsr) {
  __shared__ __align__(16) float lu[kReadoutChunk][8][8];  // [o][b mod 8][slice]
  __shared__ float wl[kAdjointRows][kReadoutChunk + 1];
  const uint32_t t = blockIdx.y, i0 = blockIdx.x * kAdjointRows;
  const uint32_t il = threadIdx.x >> 3, b8 = threadIdx.x & 7u, i = i0 + il;
  float acc[8] = {};
  // membranes of the block: [b][neuron], 32 neurons (128 bytes) contiguous
  __shared__ float vs[64][kAdjointRows + 1];
  if (a.events) {
    float v[8];
    const uint32_t n = threadIdx.x % kAdjointRows, b0 = threadIdx.x / kAdjointRows;
#pragma unroll
    for (uint32_t q = 0; q < 8; ++q) {
      const uint32_t b = b0 + 8u * q;
      v[q] = b < a.B && i0 + n < a.H ? a.vall[((size_t)t * a.B + b) * a.Hp + i0 + n] : 0.0f;
    }
#pragma unroll
    for (uint32_t q = 0; q < 8; ++q) vs[b0 + 8u * q][n] = v[q];
  }
  for (uint32_t o0 = 0; o0 < a.O; o0 += kReadoutChunk) {
    const uint32_t no = std::min<uint32_t>(kReadoutChunk, a.O - o0);
    if (o0) __syncthreads();
    for (uint32_t x = threadIdx.x; x < no * 64u; x += 256u)
      lu[x >> 6][x & 7u][(x >> 3) & 7u] = a.lamu[((size_t)t * a.O + o0) * 64 + x];
    for (uint32_t x = threadIdx.x; x < kAdjointRows * no; x += 256u) {
      const uint32_t r = x / no, o = x % no;
      wl[r][o] = i0 + r < a.H ? a.w_out[(size_t)(i0 + r) * a.O + o0 + o] : 0.0f;
    }
    __syncthreads();
    for (uint32_t o = 0; o < no; ++o) {
      const float w = wl[il][o];
      const float4 lo = *reinterpret_cast<const float4 *>(&lu[o][b8][0]);
      const float4 hi = *reinterpret_cast<const float4 *>(&lu[o][b8][4]);
      const float l[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[q] = acc[q] + w * l[q];
    }
  }
  if (i >= a.H) return;
#pragma unroll
  for (int q = 0; q < 8; ++q)
    if ((uint32_t)q < a.S) {
      const size_t at = (((size_t)t * a.S + q) * a.H + i) * 8 + b8;
      dsr[at] = acc[q];
      if (a.events) a.sg[at] = surrogate(vs[q * 8 + b8][il] - a.theta, a.slope, false);
    }
}

// x + the value of another lane of the 16-lane row, by DPP.
template <int kCtrl>
__device__ __forceinline__ float add_row_lane(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xf, 0xf, true));
}

// Sum over the 16 lanes of a row, in every lane: neighbours, pairs, then the quads and halves
// by mirroring (whose lanes already agree).
__device__ __forceinline__ float row_sum(float x) {
  x = add_row_lane<0xB1>(x);    // quad_perm 1,0,3,2
  x = add_row_lane<0x4E>(x);    // quad_perm 2,3,0,1
  x = add_row_lane<0x141>(x);   // row_half_mirror
  return add_row_lane<0x140>(x);  // row_mirror
}

// Membrane adjoint of step t in the sliced layout.  A workgroup per (slice, 32 neurons): the
// slice's lamV_{t+1} of all H neurons (32 H bytes, contiguous) is staged in LDS, requested
// together with the neurons' outgoing synapses (padded rows of (target, weight) pairs, so no
// row bounds come first) and their own state: one memory round trip.  A wavefront holds two
// neurons; of the 32 lanes of one, 16 take every 16th synapse for 4 batch elements each, one
// 16-byte LDS read and four multiply-adds per synapse, and a 16-lane sum completes them.
// Slices are dealt round-robin over the workgroups, so that with 8 slices each XCD (they
// take workgroups round-robin too) works on one slice, which its own L2 holds.  A launch and
// its round trip bound it: 4.7 us per step at 64 x 1,024 with rows of about 102 synapses
// (7.4 with a wavefront per neuron that gathers 256-byte rows from memory, the form kept for
// layers whose workgroups the device does not hold at once), 3.6 us at 19 x 201 (7.7).
// lam_next / lam_out: slices of steps t + 1 and t; lam_out holds the readout part on entry.
// v_t: V_t as [H][64], or, in the event-driven form, its surrogate derivative in the slices.
constexpr int kAdjointAhead = 8;  // rounds of synapses requested before the barrier
__global__ __launch_bounds__(1024) void k_adjoint_slice(BpttArgs a, const float *v_t, const float *lam_next,
                                                        float *lam_out) {
  extern __shared__ float4 lam_sl[];  // [H][2]
  const uint32_t slice = blockIdx.x % a.S, block = blockIdx.x / a.S;
  const uint32_t lane = lane_id(), wave = threadIdx.x / kWave;
  const uint32_t p = lane & 15u, b4 = (lane >> 4) & 1u;
  const uint32_t i = block * kAdjointRows + wave * 2u + (lane >> 5);
  const bool live = i < a.H;
  const uint32_t il = live ? i : a.H - 1u;
  const uint2 *row = a.adj_pair + (size_t)il * a.adj_w;
  const uint32_t len = live ? a.adj_len[il] : 0u;
  uint2 e[kAdjointAhead];
#pragma unroll
  for (int k = 0; k < kAdjointAhead; ++k) {
    e[k] = make_uint2(0u, 0u);
    if ((uint32_t)k * 16u < a.adj_w) e[k] = row[(uint32_t)k * 16u + p];  // uniform condition
  }
  // this lane's element of the result (p < 4): batch element b
  const uint32_t b = slice * 8u + b4 * 4u + (p & 3u);
  const size_t own = ((size_t)slice * a.H + il) * 8 + (b & 7u);
  const float ln = lam_next[own], readout = lam_out[own];
  const float vt = a.events ? v_t[own] : v_t[(size_t)il * 64 + b];
  const float4 *src = reinterpret_cast<const float4 *>(lam_next + (size_t)slice * a.H * 8);
  for (uint32_t x0 = threadIdx.x; x0 < a.H * 2u; x0 += 4u * 1024u) {
    float4 v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = src[std::min<uint32_t>(x0 + (uint32_t)q * 1024u, a.H * 2u - 1u)];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (x0 + (uint32_t)q * 1024u < a.H * 2u) lam_sl[x0 + (uint32_t)q * 1024u] = v[q];
  }
  __syncthreads();
  float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  // (a padding entry is skipped, not multiplied: its target's adjoint may not be finite)
  auto add = [&](const uint2 &s, uint32_t at) {
    const float4 l = lam_sl[s.x * 2u + b4];
    const float w = __uint_as_float(s.y);
    if (at < len) {
      acc.x = __builtin_fmaf(w, l.x, acc.x);
      acc.y = __builtin_fmaf(w, l.y, acc.y);
      acc.z = __builtin_fmaf(w, l.z, acc.z);
      acc.w = __builtin_fmaf(w, l.w, acc.w);
    }
  };
#pragma unroll
  for (int k = 0; k < kAdjointAhead; ++k)
    if ((uint32_t)k * 16u < a.adj_w) add(e[k], (uint32_t)k * 16u + p);
  for (uint32_t at = kAdjointAhead * 16u + p; at < a.adj_w; at += 16u) add(row[at], at);
  acc.x = row_sum(acc.x);
  acc.y = row_sum(acc.y);
  acc.z = row_sum(acc.z);
  acc.w = row_sum(acc.w);
  if (!live || p >= 4u) return;
  const float sum = p == 0 ? acc.x : p == 1 ? acc.y : p == 2 ? acc.z : acc.w;
  float ds = readout + sum;
  if (!a.detach_reset) ds = ds - a.theta * ln;
  const float g = a.events ? vt : surrogate(vt - a.theta, a.slope, a.smooth != 0);
  lam_out[own] = a.beta * ln + g * ds;
}

// ---- the membrane adjoint of one batch element in one workgroup ---------------------------
// Batch elements do not interact in the membrane adjoint either.  Where the synapses fit the
// registers and the LDS of a compute unit, a workgroup runs all steps of one element:
// lamV_{t+1} of all neurons sits in LDS, and seq_p lanes share a neuron's row of W_rec.  A
// lane's synapses keep their places for the whole pass, the first kRegs of them in registers
// (a weight, and an LDS offset in 16 bits), the others in LDS.  The plan orders a lane's
// synapses so that the 32 lanes that read LDS together meet few bank conflicts, and deals
// rows to lanes by length, so that a wavefront's lanes carry equally many.  Places without a
// synapse read a zero that follows the neurons.  One barrier per step; no step waits for a
// launch: 0.5 us per step at 201 neurons (3.6 launched), 2.5 at 700 with 70 synapses each
// (about 4).  104,000 synapses at 1,024 neurons do not fit; a variant that streamed what did
// not fit from L2 took 6.2 us per step, against 4.7 launched.
constexpr int kSeqState = 4;  // steps of (readout part, surrogate) requested ahead
template <int kRegs>
__global__ __launch_bounds__(1024) void k_adjoint_seq(BpttArgs a) {
  extern __shared__ float4 more_s[];  // the places past kRegs: weights, then offsets
  __shared__ float lam_s[2][kSeqMaxNeurons + 1];
  // the 8 elements of a slice run on one XCD (workgroups are dealt round-robin), whose L2
  // merges their 4-byte reads and writes of the slice's lines
  const uint32_t b = a.S == 8 ? (blockIdx.x & 7u) * 8u + (blockIdx.x >> 3) : blockIdx.x;
  if (b >= a.B) return;
  const uint32_t tid = threadIdx.x, n_thr = a.seq_threads, lane = lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const uint32_t row = a.seq_row[tid];
  const bool owner = row != 0xFFFFFFFFu && (tid & (a.seq_p - 1u)) == 0;  // stores the row's result
  const uint32_t i = row != 0xFFFFFFFFu ? row : 0u;
  const uint32_t groups = a.seq_groups[wave];    // groups of four places, of them in LDS:
  const uint32_t more = groups > kRegs / 4 ? groups - kRegs / 4 : 0u;
  const float4 *wg = reinterpret_cast<const float4 *>(a.seq_w) + tid;
  const uint2 *cg = reinterpret_cast<const uint2 *>(a.seq_col) + tid;
  float4 w[kRegs / 4];
  uint2 c[kRegs / 4];
#pragma unroll
  for (int g = 0; g < kRegs / 4; ++g) {
    w[g] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    c[g] = make_uint2(0u, 0u);
    if ((uint32_t)g < groups) {
      w[g] = wg[(size_t)g * n_thr];
      c[g] = cg[(size_t)g * n_thr];
    }
  }
  float4 *w_more = more_s + a.seq_more[wave] * kWave + lane;
  uint2 *c_more = reinterpret_cast<uint2 *>(more_s + a.seq_more_all * kWave) + a.seq_more[wave] * kWave + lane;
  for (uint32_t g = 0; g < more; ++g) {  // a lane reads back only what it wrote
    w_more[g * kWave] = wg[(size_t)(kRegs / 4 + g) * n_thr];
    c_more[g * kWave] = cg[(size_t)(kRegs / 4 + g) * n_thr];
  }
  const size_t slices = (size_t)a.S * a.H * 8, own = ((size_t)(b >> 3) * a.H + i) * 8 + (b & 7u);
  float *lam_out = a.lamv + own;
  const float *sg = a.sg + own;
  float ln = 0.0f, ro_t[kSeqState], sg_t[kSeqState];
#pragma unroll
  for (int q = 0; q < kSeqState; ++q) {
    const uint32_t t = a.T - 1u - std::min<uint32_t>((uint32_t)q, a.T - 1u);
    ro_t[q] = lam_out[t * slices];
    sg_t[q] = sg[t * slices];
  }
  for (uint32_t x = tid; x < 2 * (kSeqMaxNeurons + 1); x += blockDim.x) (&lam_s[0][0])[x] = 0.0f;
  __syncthreads();
  auto add4 = [&](float4 &acc, const float4 &wv, const uint2 &cv, const char *l) {
    acc.x = __builtin_fmaf(wv.x, *reinterpret_cast<const float *>(l + (cv.x & 0xFFFFu)), acc.x);
    acc.y = __builtin_fmaf(wv.y, *reinterpret_cast<const float *>(l + (cv.x >> 16)), acc.y);
    acc.z = __builtin_fmaf(wv.z, *reinterpret_cast<const float *>(l + (cv.y & 0xFFFFu)), acc.z);
    acc.w = __builtin_fmaf(wv.w, *reinterpret_cast<const float *>(l + (cv.y >> 16)), acc.w);
  };
  for (uint32_t n0 = 0; n0 < a.T; n0 += kSeqState) {
#pragma unroll
    for (int q = 0; q < kSeqState; ++q) {
      if (n0 + (uint32_t)q < a.T) {  // uniform
        const uint32_t t = a.T - 1u - (n0 + (uint32_t)q);
        const char *l = reinterpret_cast<const char *>(&lam_s[q & 1][0]);  // kSeqState is even
        float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
        for (int g = 0; g < kRegs / 4; ++g)
          if ((uint32_t)g < groups) add4(acc, w[g], c[g], l);
        if (more) {
          float4 wn = w_more[0];
          uint2 cn = c_more[0];
          for (uint32_t g = 0; g < more; ++g) {
            const float4 wv = wn;
            const uint2 cv = cn;
            const uint32_t nx = std::min<uint32_t>(g + 1u, more - 1u);
            wn = w_more[nx * kWave];
            cn = c_more[nx * kWave];
            add4(acc, wv, cv, l);
          }
        }
        float sum = (acc.x + acc.y) + (acc.z + acc.w);
        if (a.seq_p >= 2) sum = add_row_lane<0xB1>(sum);
        if (a.seq_p >= 4) sum = add_row_lane<0x4E>(sum);
        if (a.seq_p >= 8) sum = add_row_lane<0x141>(sum);
        if (a.seq_p >= 16) sum = add_row_lane<0x140>(sum);
        float ds = ro_t[q] + sum;
        if (!a.detach_reset) ds = ds - a.theta * ln;
        ln = a.beta * ln + sg_t[q] * ds;
        // the state of kSeqState steps ahead
        const uint32_t t_next = t >= (uint32_t)kSeqState ? t - kSeqState : 0u;
        ro_t[q] = lam_out[t_next * slices];
        sg_t[q] = sg[t_next * slices];
        if (owner) {
          lam_s[(q & 1) ^ 1][i] = ln;
          lam_out[t * slices] = ln;
        }
        __syncthreads();
      }
    }
  }
}

// Batch masks of a [T][rows][64] trajectory: bits[r][t] bit b = (val[t][r][b] != 0) for
// b < B; flag receives 1 if any of those values is neither 0 nor 1 (the masks then do
// not represent the values and the gradients take the general path).  A wavefront per
// (t, r).
__global__ __launch_bounds__(256) void k_bits(const float *val, uint32_t rows, uint32_t T, uint32_t B,
                                              uint64_t *bits, uint32_t *flag) {
  const uint64_t w = (uint64_t)blockIdx.x * 4 + threadIdx.x / kWave;
  if (w >= (uint64_t)T * rows) return;
  const uint32_t t = (uint32_t)(w / rows), r = (uint32_t)(w % rows), b = lane_id();
  const float x = val[w * 64 + b];
  const bool on = b < B && x != 0.0f;
  const uint64_t m = __ballot(on);
  const uint64_t bad = __ballot(on && x != 1.0f);
  if (b == 0) {
    bits[(size_t)r * T + t] = m;
    if (bad) atomicOr(flag, 1u);
  }
}

constexpr uint32_t kXcdCount = 8;  // XCDs take workgroups round-robin
constexpr int kGradBlock = 256;
constexpr uint32_t kGradChunk = 128;  // steps of lamV staged in LDS at a time (32 KB)
constexpr int kMaskAhead = 8;         // mask words in flight per lane

// Gradients of the sparse weights, one owner per synapse: the adjoint of the current
// I_t = W_in^T x_t + W_rec^T s_{t-1} gives
//   g_in[c -> j]  = sum_t sum_b x_t[c][b] lamV_t[j][b]
//   g_rec[i -> j] = sum_t sum_b s_{t-1}[i][b] lamV_t[j][b].
// One workgroup per target j stages lamV_t[j][.] in LDS, kGradChunk steps at a time; each
// lane owns one in-edge of j (input projection first, then recurrent, each in ascending
// source order), kGradBlock edges per pass.  With binary presynaptic values (the masks'
// flag clear) the lane walks the set bits of its source's batch mask of every step and
// adds the matching lamV entries in ascending b, summing each step before adding it to
// the edge's total; otherwise it multiplies the stored values in.  The mask words of the
// next kMaskAhead steps are loaded while the current ones are used.
__global__ __launch_bounds__(kGradBlock) void k_grad_edges(BpttArgs a, const uint64_t *xbits,
                                                           const uint64_t *sbits, const uint32_t *flags) {
  extern __shared__ float lam_s[];  // [kGradChunk][64]
  const uint32_t j = blockIdx.x;
  const uint64_t in0 = a.in_t_ptr[j], rec0 = a.rec_t_ptr[j];
  const uint32_t n_in = (uint32_t)(a.in_t_ptr[j + 1] - in0), n_rec = (uint32_t)(a.rec_t_ptr[j + 1] - rec0);
  const uint32_t deg = n_in + n_rec, T = a.T;
  const bool x_bits = flags[0] == 0, s_bits = !a.smooth && flags[1] == 0;
  for (uint32_t base = 0; base < deg; base += kGradBlock) {
    const uint32_t k = base + threadIdx.x;
    const bool live = k < deg, is_in = k < n_in;
    uint32_t src = 0, edge = 0;
    if (live) {
      src = (uint32_t)(is_in ? a.in_t_src[in0 + k] : a.rec_t_src[rec0 + (k - n_in)]);
      edge = is_in ? a.in_t_edge[in0 + k] : a.rec_t_edge[rec0 + (k - n_in)];
    }
    const bool use_bits = is_in ? x_bits : s_bits;
    // the lane's mask row: the input's step t, or the hidden neuron's step t - 1
    const uint64_t *row = is_in ? xbits + (size_t)src * T : sbits + (size_t)src * T;
    const uint32_t lag = is_in ? 0u : 1u;
    auto mask_at = [&](uint32_t t) -> uint64_t {
      return (live && use_bits && t >= lag && t - lag < T) ? row[t - lag] : 0ull;
    };
    float total = 0.0f;
    for (uint32_t tc = 0; tc < T; tc += kGradChunk) {
      const uint32_t len = min(kGradChunk, T - tc);
      __syncthreads();  // the previous chunk has been read by every lane
      for (uint32_t x = threadIdx.x; x < len * 64; x += kGradBlock) {
        const uint32_t t = tc + x / 64, b = x & 63u;
        if (a.S) lam_s[x] = b < a.S * 8u ? a.lamv[slice_index(a, t, b, j)] : 0.0f;
        else lam_s[x] = a.lamv[((size_t)t * a.H + j) * 64 + b];
      }
      __syncthreads();
      if (!live) continue;
      if (use_bits) {
        uint64_t cur[kMaskAhead], nxt[kMaskAhead];
#pragma unroll
        for (int q = 0; q < kMaskAhead; ++q) cur[q] = mask_at(tc + q);
        for (uint32_t u0 = 0; u0 < len; u0 += kMaskAhead) {
#pragma unroll
          for (int q = 0; q < kMaskAhead; ++q) nxt[q] = u0 + kMaskAhead + q < len ? mask_at(tc + u0 + kMaskAhead + q) : 0ull;
#pragma unroll
          for (int q = 0; q < kMaskAhead; ++q) {
            if (u0 + q >= len) break;
            uint64_t m = cur[q];
            const float *lt = lam_s + (size_t)(u0 + q) * 64;
            float part = 0.0f;
            while (m) {
              part += lt[__builtin_ctzll(m)];
              m &= m - 1;
            }
            total += part;
          }
#pragma unroll
          for (int q = 0; q < kMaskAhead; ++q) cur[q] = nxt[q];
        }
      } else {
        for (uint32_t u = 0; u < len; ++u) {
          const uint32_t t = tc + u;
          if (t < lag) continue;
          const float *val = is_in ? a.xt + ((size_t)t * a.C + src) * 64 : a.s + ((size_t)(t - 1) * a.H + src) * 64;
          const float *lt = lam_s + (size_t)u * 64;
          float part = 0.0f;
          for (uint32_t b = 0; b < a.B; ++b) part += val[b] * lt[b];
          total += part;
        }
      }
    }
    if (live) (is_in ? a.g_w_in : a.g_w_rec)[edge] = total;
  }
}

// ---- sparse-weight gradients from event lists (the event-driven form) ------------------------
// A source's events of a chunk of kListChunk steps, as 16-bit indices into the chunk's
// lamV_t[b] values ((t - t_chunk) 64 + b, ascending), padded to whole groups of 8 with the
// index of a zero: lanes that walk lists of their own diverge only in the lists' lengths,
// where lanes that walk 64-bit masks step by step wait for the busiest lane in every step.
constexpr uint32_t kListChunk = 128;
constexpr uint32_t kListCap = kListChunk * 64 / 4;  // events of a list: a quarter of the chunk
constexpr uint32_t kListStride = kListCap + 8;      // one group is read ahead
constexpr uint32_t kListZero = kListChunk * 64;

// Lists of the inputs (sources 0 .. C - 1, step t) and of the hidden neurons (C .. C + H - 1,
// step t - 1); a wavefront per (source, chunk).  A source with more than kListCap events in
// the chunk gets its count only.
__global__ __launch_bounds__(256) void k_event_lists(BpttArgs a) {
  const uint32_t w = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t n_chunks = (a.T + kListChunk - 1) / kListChunk;
  if (w >= (a.C + a.H) * n_chunks) return;
  const uint32_t r = w / n_chunks, c = w % n_chunks, lane = lane_id();
  const bool is_in = r < a.C;
  const uint64_t *row = is_in ? a.xbits + (size_t)r * a.T : a.sbits + (size_t)(r - a.C) * a.T;
  const uint32_t lag = is_in ? 0u : 1u;
  uint16_t *list = a.lists + (size_t)w * kListStride;
  uint64_t m[kListChunk / 64];
#pragma unroll
  for (uint32_t h = 0; h < kListChunk / 64; ++h) {
    const uint32_t t = c * kListChunk + h * 64u + lane;
    m[h] = t < a.T && t >= lag ? row[t - lag] : 0ull;
  }
  uint32_t n = 0, at[kListChunk / 64];
#pragma unroll
  for (uint32_t h = 0; h < kListChunk / 64; ++h) {
    const uint32_t p = (uint32_t)__popcll(m[h]), incl = wave_inclusive_scan(p);
    at[h] = n + incl - p;
    n += (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
  }
  if (lane == 0) a.list_len[w] = n;
  if (n > kListCap) return;
#pragma unroll
  for (uint32_t h = 0; h < kListChunk / 64; ++h)
    for (uint64_t x = m[h]; x; x &= x - 1) list[at[h]++] = (uint16_t)((h * 64u + lane) * 64u + (uint32_t)__builtin_ctzll(x));
  if (lane < ((0u - n) & 7u)) list[n + lane] = (uint16_t)kListZero;
}

// One owner per synapse, as k_grad_edges: a workgroup per target j stages lamV_t[j][.] of a
// chunk in LDS; a lane owns up to kListEdges in-edges and adds the values at its source's
// events, eight per 16-byte list read, in four sums.  Targets are numbered so that four
// neighbours, whose slices share cache lines, run on one XCD one after another.  Bound: the
// LDS reads, of the longest list in each wavefront.  248,000 edges of 64 x 250, 700 -> 1,024:
// 65 us and 5 us of lists, where walking the masks took 263.
constexpr int kListEdges = 4;
__global__ __launch_bounds__(kGradBlock) void k_grad_lists(BpttArgs a) {
  __shared__ float lam_c[kListChunk * 64 + 1];
  const uint32_t g = blockIdx.x / kXcdCount;
  const uint32_t j = ((g >> 2) * kXcdCount + blockIdx.x % kXcdCount) * 4u + (g & 3u);
  if (j >= a.H) return;
  const uint64_t in0 = a.in_t_ptr[j], rec0 = a.rec_t_ptr[j];
  const uint32_t n_in = (uint32_t)(a.in_t_ptr[j + 1] - in0), n_rec = (uint32_t)(a.rec_t_ptr[j + 1] - rec0);
  const uint32_t deg = n_in + n_rec, n_chunks = (a.T + kListChunk - 1) / kListChunk;
  const bool x_bits = a.flags[0] == 0;
  if (threadIdx.x == 0) lam_c[kListZero] = 0.0f;
  for (uint32_t base = 0; base < deg; base += kGradBlock * kListEdges) {
    float total[kListEdges];
    uint32_t src[kListEdges];
#pragma unroll
    for (int p = 0; p < kListEdges; ++p) {
      const uint32_t k = base + (uint32_t)p * kGradBlock + threadIdx.x;
      total[p] = 0.0f;
      src[p] = k < n_in ? (uint32_t)a.in_t_src[in0 + k] : k < deg ? a.C + (uint32_t)a.rec_t_src[rec0 + (k - n_in)] : 0u;
    }
    for (uint32_t c = 0; c < n_chunks; ++c) {
      const uint32_t tc = c * kListChunk, len = min(kListChunk, a.T - tc);
      __syncthreads();  // the previous chunk has been read by every lane
      for (uint32_t x0 = threadIdx.x; x0 < len * 64; x0 += 8 * kGradBlock) {
        float v[8];
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) {
          const uint32_t x = std::min<uint32_t>(x0 + q * kGradBlock, len * 64 - 1), b = x & 63u;
          v[q] = b < a.S * 8u ? a.lamv[slice_index(a, tc + (x >> 6), b, j)] : 0.0f;
        }
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q)
          if (x0 + q * kGradBlock < len * 64) lam_c[x0 + q * kGradBlock] = v[q];
      }
      __syncthreads();
#pragma unroll
      for (int p = 0; p < kListEdges; ++p) {
        const uint32_t k = base + (uint32_t)p * kGradBlock + threadIdx.x;
        if (k >= deg) continue;
        const bool is_in = k < n_in;
        if (is_in && !x_bits) {  // inputs other than 0 and 1
          for (uint32_t u = 0; u < len; ++u) {
            const float *val = a.xt + ((size_t)(tc + u) * a.C + src[p]) * 64, *lt = lam_c + u * 64;
            float part = 0.0f;
            for (uint32_t b = 0; b < a.B; ++b) part += val[b] * lt[b];
            total[p] += part;
          }
          continue;
        }
        const size_t id = (size_t)src[p] * n_chunks + c;
        const uint32_t n = a.list_len[id];
        if (n > kListCap) {  // too many events for a list: the masks
          const uint32_t lag = is_in ? 0u : 1u;
          const uint64_t *row = is_in ? a.xbits + (size_t)src[p] * a.T : a.sbits + (size_t)(src[p] - a.C) * a.T;
          for (uint32_t u = tc < lag ? 1u : 0u; u < len; ++u) {
            float part = 0.0f;
            for (uint64_t m = row[tc + u - lag]; m; m &= m - 1) part += lam_c[u * 64 + (uint32_t)__builtin_ctzll(m)];
            total[p] += part;
          }
          continue;
        }
        const uint4 *list = reinterpret_cast<const uint4 *>(a.lists + id * kListStride);
        float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
        uint4 e = list[0];
        for (uint32_t q = 0; q < n; q += 8) {
          const uint4 nx = list[q / 8 + 1];
          s0 += lam_c[e.x & 0xFFFFu];
          s1 += lam_c[e.x >> 16];
          s2 += lam_c[e.y & 0xFFFFu];
          s3 += lam_c[e.y >> 16];
          s0 += lam_c[e.z & 0xFFFFu];
          s1 += lam_c[e.z >> 16];
          s2 += lam_c[e.w & 0xFFFFu];
          s3 += lam_c[e.w >> 16];
          e = nx;
        }
        total[p] += (s0 + s1) + (s2 + s3);
      }
    }
#pragma unroll
    for (int p = 0; p < kListEdges; ++p) {
      const uint32_t k = base + (uint32_t)p * kGradBlock + threadIdx.x;
      if (k < n_in) a.g_w_in[a.in_t_edge[in0 + k]] = total[p];
      else if (k < deg) a.g_w_rec[a.rec_t_edge[rec0 + (k - n_in)]] = total[p];
    }
  }
}

// Gradient of the dense readout weights over the whole sequence: one wavefront per
// hidden neuron i and output o; four partial sums keep loads of later steps in flight.
__global__ __launch_bounds__(256) void k_grad_out(BpttArgs a) {
  const uint32_t w = blockIdx.x * 4 + threadIdx.x / kWave;
  if (w >= a.H * a.O) return;
  const uint32_t i = w / a.O, o = w % a.O, b = lane_id();
  const float *sp = a.s + (size_t)i * 64 + b;
  const float *lp = a.lamu + (size_t)o * 64 + b;
  const size_t ss = (size_t)a.H * 64, ls = (size_t)a.O * 64;
  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  uint32_t t = 0;
  for (; t + 4 <= a.T; t += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] += sp[(t + u) * ss] * lp[(t + u) * ls];
  }
  for (; t < a.T; ++t) acc[0] += sp[t * ss] * lp[t * ls];
  const float sum = wave_sum((acc[0] + acc[1]) + (acc[2] + acc[3]));
  if (b == 0) a.g_w_out[(size_t)i * a.O + o] = sum;
}

// The same from the spike masks: a wavefront per (neuron, block of kOutBlock readouts) visits
// the steps at which the neuron spikes in some batch element and adds the readout adjoints of
// the lanes (batch elements) that spike.  With an adjoint that is not finite it visits every step
// and multiplies, as the sum is defined.
constexpr int kOutBlock = 4;
constexpr int kOutSteps = 8;
__global__ __launch_bounds__(256) void k_grad_out_events(BpttArgs a) {
  const uint32_t n_blocks = (a.O + kOutBlock - 1) / kOutBlock;
  const uint32_t w = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (w >= a.H * n_blocks) return;
  const uint32_t i = w / n_blocks, o0 = w % n_blocks * kOutBlock, lane = lane_id();
  const uint32_t no = std::min<uint32_t>(kOutBlock, a.O - o0);
  float acc[kOutBlock] = {};
  const bool every = a.flags[3] != 0;
  for (uint32_t t0 = 0; t0 < a.T; t0 += kWave) {
    const uint64_t mine = t0 + lane < a.T ? a.sbits[(size_t)i * a.T + t0 + lane] : 0ull;
    // kOutSteps steps requested together (the last one again where fewer are left, unused)
    uint64_t any = __ballot(mine != 0);
    while (any) {
      float l[kOutSteps][kOutBlock];
      uint64_t on[kOutSteps];
      uint32_t k = 0;
#pragma unroll
      for (int u = 0; u < kOutSteps; ++u) {
        const bool more = any != 0;  // uniform
        if (more) k = (uint32_t)__builtin_ctzll(any);
        any &= any - 1;
        on[u] = more ? lane_read64(mine, k) : 0ull;
        const float *lu = a.lamu + ((size_t)(t0 + k) * a.O + o0) * 64 + lane;
#pragma unroll
        for (int q = 0; q < kOutBlock; ++q) l[u][q] = lu[std::min<uint32_t>(q, no - 1) * 64];
      }
#pragma unroll
      for (int u = 0; u < kOutSteps; ++u) {
        const bool mine_on = __builtin_amdgcn_inverse_ballot_w64(on[u]);
#pragma unroll
        for (int q = 0; q < kOutBlock; ++q) acc[q] += mine_on ? l[u][q] : 0.0f;
      }
    }
  }
  if (every) {
#pragma unroll
    for (int q = 0; q < kOutBlock; ++q) acc[q] = 0.0f;
    for (uint32_t t = 0; t < a.T; ++t) {
      const float on = (a.sbits[(size_t)i * a.T + t] >> lane) & 1u ? 1.0f : 0.0f;
#pragma unroll
      for (int q = 0; q < kOutBlock; ++q)
        acc[q] += on * a.lamu[((size_t)t * a.O + o0 + std::min<uint32_t>(q, no - 1)) * 64 + lane];
    }
  }
#pragma unroll
  for (int q = 0; q < kOutBlock; ++q) {
    const float sum = wave_sum(acc[q]);
    if (lane == 0 && (uint32_t)q < no) a.g_w_out[(size_t)i * a.O + o0 + q] = sum;
  }
}

__global__ void k_fill(float *p, uint64_t n, float v) {
  const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < n) p[idx] = v;
}

uint32_t blocks_for(uint64_t n, uint32_t per) { return (uint32_t)((n + per - 1) / per); }

}  // namespace

// ELL-order copy of the recurrent weights: w_ell[x] = w[edge[x]], 0 for padding.
__global__ void k_gather_ell(const float *w, const uint32_t *edge, float *w_ell, uint64_t n) {
  const uint64_t x = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x < n) w_ell[x] = edge[x] == 0xFFFFFFFFu ? 0.0f : w[edge[x]];
}

// The layouts' index arrays, a wavefront per neuron: its in-edges of both projections and its row.
__global__ __launch_bounds__(256) void k_fill_layouts(BpttArgs a, BpttLayouts lay) {
  const uint32_t j = blockIdx.x * 4 + threadIdx.x / kWave, lane = lane_id();
  if (j >= a.H) return;
  if (lay.in_pos)
    for (uint64_t x = a.in_t_ptr[j] + lane; x < a.in_t_ptr[j + 1]; x += kWave)
      lay.in_pos[a.in_t_edge[x]] = (uint32_t)a.in_t_src[x] * a.Hp + j;
  const uint64_t e0 = a.rec_t_ptr[j];
  const uint32_t n_in = (uint32_t)(a.rec_t_ptr[j + 1] - e0);
  if (lay.rec_pos)
    for (uint32_t k = lane; k < n_in; k += kWave) {
      const uint32_t src = (uint32_t)a.rec_t_src[e0 + k], edge = a.rec_t_edge[e0 + k];
      lay.rec_pos[edge] = src * a.Hp + j;
      lay.col_pos[edge] = k * a.Hp + j;
      a.col_pair[(size_t)k * a.Hp + j].x = src;
    }
  if (lay.ell_src) {  // padding: source 0, edge 0xFFFFFFFF
    const size_t row = (size_t)j * a.ell_w;
    for (uint32_t k = lane; k < a.ell_w; k += kWave) {
      lay.ell_src[row + k] = k < n_in ? a.rec_t_src[e0 + k] : 0;
      lay.ell_edge[row + k] = k < n_in ? a.rec_t_edge[e0 + k] : 0xFFFFFFFFu;
    }
    if (lane == 0) lay.ell_len[j] = n_in;
  }
  if (lay.adj_pos) {
    const uint64_t r0 = a.rec_ptr[j];
    const uint32_t n_out = (uint32_t)(a.rec_ptr[j + 1] - r0);
    for (uint32_t k = lane; k < n_out; k += kWave) {
      lay.adj_pos[r0 + k] = j * a.adj_w + k;
      a.adj_pair[(size_t)j * a.adj_w + k].x = (uint32_t)a.rec_col[r0 + k];
    }
    if (lane == 0) lay.adj_len[j] = n_out;
  }
}

// The weights of the sliced adjoint's padded rows: edge e of the CSR order at pos[e].
__global__ void k_scatter_pairs(const float *w, const uint32_t *pos, uint2 *pair, uint64_t nnz) {
  const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < nnz) pair[pos[e]].y = __float_as_uint(w[e]);
}

__global__ void k_scatter_rows(const float *w, const uint32_t *pos, float *rows, uint64_t nnz) {
  const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < nnz) rows[pos[e]] = w[e];
}

static void gather_weights(const BpttArgs &a, hipStream_t s) {
  if (a.ell_w)
    hipLaunchKernelGGL(k_gather_ell, dim3(blocks_for((uint64_t)a.H * a.ell_w, 256)), dim3(256), 0, s, a.w_rec,
                       a.ell_edge, a.ell_wt, (uint64_t)a.H * a.ell_w);
  if (a.nnz_in)
    hipLaunchKernelGGL(k_gather_t, dim3(blocks_for(a.nnz_in, 256)), dim3(256), 0, s, a.w_in, a.in_t_edge,
                       a.w_in_t, a.nnz_in);
  if (a.nnz_rec)
    hipLaunchKernelGGL(k_gather_t, dim3(blocks_for(a.nnz_rec, 256)), dim3(256), 0, s, a.w_rec, a.rec_t_edge,
                       a.w_rec_t, a.nnz_rec);
}

// The forward and backward passes each run as three parts.  The prologue and epilogue
// read or write the caller's arrays (inputs, weights, labels, loss, gradients); the body
// in between touches only the plan's own buffers (its weight copies included), so the
// runtime can capture it once per plan in a HIP graph and replay it on every call.

hipError_t bptt_forward_prologue(const BpttArgs &a, const float *x, bool busy, hipStream_t s) {
  if (a.events) {
    const uint64_t nnz = std::max<uint64_t>(std::max(a.nnz_in, a.nnz_rec), 3);
    hipLaunchKernelGGL(k_scatter_weights, dim3(blocks_for(nnz, 256)), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_transpose_x, dim3((a.C + 63) / 64, a.T), dim3(256), 0, s, x, a.xt, a.xbits, a.flags, a.B,
                       a.T, a.C, a.w_out, a.H * a.O);
    if (busy) {
      gather_weights(a, s);
      hipLaunchKernelGGL(k_input_current, dim3(blocks_for((uint64_t)((a.T + kMaskSteps - 1) / kMaskSteps) * a.H, 4)),
                         dim3(256), 0, s, a);
    } else {
      hipLaunchKernelGGL(k_input_rows, dim3(blocks_for((uint64_t)a.B * a.T, 4), blocks_for(a.Hp / 256, kInputBlocks)),
                         dim3(256), 0, s, a, x);
    }
    hipLaunchKernelGGL(k_input_current_values, dim3(std::min<uint32_t>(blocks_for((uint64_t)a.T * a.H, 4), kValuesGrid)),
                       dim3(256), 0, s, a, busy);
    return hipGetLastError();
  }
  gather_weights(a, s);
  // flags[0] is set below if some input is neither 0 nor 1; flags[1] only by the backward
  // pass of a smooth-mode plan
  hipLaunchKernelGGL(k_fill, dim3(1), dim3(64), 0, s, reinterpret_cast<float *>(a.flags), (uint64_t)2, 0.0f);
  hipLaunchKernelGGL(k_transpose_x, dim3((a.C + 63) / 64, a.T), dim3(256), 0, s, x, a.xt, a.xbits, a.flags, a.B,
                     a.T, a.C, a.w_out, 0u);
  const hipError_t e = hipMemcpyAsync(a.w_out_c, a.w_out, (size_t)a.H * a.O * 4, hipMemcpyDeviceToDevice, s);
  return e != hipSuccess ? e : hipGetLastError();
}

// The spike masks of the latest event-driven forward pass, for the backward pass and the trace.
hipError_t bptt_spike_masks(const BpttArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_spike_masks, dim3(a.nw, blocks_for(a.T, kMaskBlock)), dim3(256), 0, s, a);
  return hipGetLastError();
}

// The hidden steps of the event-driven form, one workgroup per batch element.
hipError_t bptt_hidden_seq(const BpttArgs &a, hipStream_t s) {
  // whole wavefronts up to Hp, a multiple of 256
  const size_t lds = (size_t)kSeqChunk * a.Hp * sizeof(float);
  if (a.Hp <= 256) hipLaunchKernelGGL(k_hidden_seq<1>, dim3(a.B), dim3(a.Hp), lds, s, a);
  else if (a.Hp <= 1024) hipLaunchKernelGGL(k_hidden_seq<2>, dim3(a.B), dim3(a.Hp / 2), lds, s, a);
  else hipLaunchKernelGGL(k_hidden_seq<4>, dim3(a.B), dim3(a.Hp / 4), lds, s, a);
  return hipGetLastError();
}

// ... and its readout, after either form of the hidden steps.
hipError_t bptt_readout_events(const BpttArgs &a, bool busy, hipStream_t s) {
  if (busy) hipLaunchKernelGGL(k_readout_masks, dim3(a.T, blocks_for(a.O, kMaskOuts)), dim3(64), 0, s, a, a.ro);
  else hipLaunchKernelGGL(k_readout_events, dim3(blocks_for((uint64_t)a.B * a.T, 4)), dim3(256), 0, s, a, a.ro);
  hipLaunchKernelGGL(k_readout_scan_events, dim3(a.B + 2, blocks_for(a.O, 64)), dim3(64), 0, s, a, a.ro);
  return hipGetLastError();
}

// g: the plan's arguments with w_out = w_out_c
hipError_t bptt_forward_body(const BpttArgs &g, hipStream_t s) {
  if (g.events) {  // the hidden steps of the busy form
    const dim3 grid(blocks_for(g.H, 4));
    const size_t lds = (size_t)g.H * sizeof(uint64_t);
    for (uint32_t t = 0; t < g.T; ++t) {
      switch (g.ell_w / kWave) {
        case 0: hipLaunchKernelGGL(k_hidden_step_busy<0>, grid, dim3(256), lds, s, g, t); break;
        case 1: hipLaunchKernelGGL(k_hidden_step_busy<1>, grid, dim3(256), lds, s, g, t); break;
        case 2: hipLaunchKernelGGL(k_hidden_step_busy<2>, grid, dim3(256), lds, s, g, t); break;
        case 3: hipLaunchKernelGGL(k_hidden_step_busy<3>, grid, dim3(256), lds, s, g, t); break;
        default: hipLaunchKernelGGL(k_hidden_step_busy<4>, grid, dim3(256), lds, s, g, t); break;
      }
    }
    hipLaunchKernelGGL(k_busy_rows, dim3(g.nw, g.T), dim3(256), 0, s, g);
    return hipGetLastError();
  }
  // the inputs' batch masks and flags[0] come from the prologue's transpose
  hipLaunchKernelGGL(k_input_current, dim3(blocks_for((uint64_t)((g.T + kMaskSteps - 1) / kMaskSteps) * g.H, 4)),
                     dim3(256), 0, s, g);
  hipLaunchKernelGGL(k_input_current_values, dim3(std::min<uint32_t>(blocks_for((uint64_t)g.T * g.H, 4), kValuesGrid)),
                     dim3(256), 0, s, g, false);
  const dim3 grid(blocks_for(g.H, 4));
  float *vprev = nullptr;
  for (uint32_t t = 0; t < g.T; ++t) {
    // V of the step before each checkpoint segment is kept; the others rotate
    float *v_out = (t % g.K == g.K - 1 || t == g.T - 1) ? g.vck + (size_t)(t / g.K) * g.H * 64
                                                          : g.vtmp + (size_t)(t & 1u) * g.H * 64;
    const float *sprev = t ? g.s + (size_t)(t - 1) * g.H * 64 : nullptr;
    float *s_out = g.s + (size_t)t * g.H * 64;
    if (!g.smooth && g.ell_w) {
      const size_t lds = (size_t)g.H * sizeof(uint64_t);
      switch (g.ell_w / kWave) {
        case 1: hipLaunchKernelGGL(k_hidden_step_ell<1>, grid, dim3(256), lds, s, g, t, vprev, sprev, v_out, s_out); break;
        case 2: hipLaunchKernelGGL(k_hidden_step_ell<2>, grid, dim3(256), lds, s, g, t, vprev, sprev, v_out, s_out); break;
        case 3: hipLaunchKernelGGL(k_hidden_step_ell<3>, grid, dim3(256), lds, s, g, t, vprev, sprev, v_out, s_out); break;
        default: hipLaunchKernelGGL(k_hidden_step_ell<4>, grid, dim3(256), lds, s, g, t, vprev, sprev, v_out, s_out); break;
      }
    } else {
      hipLaunchKernelGGL(k_hidden_step, grid, dim3(256), 0, s, g, t, vprev, sprev, v_out, s_out);
    }
    vprev = v_out;
  }
  hipLaunchKernelGGL(k_readout_drive, dim3(blocks_for((uint64_t)g.T * g.O * 64, 256)), dim3(256), 0, s, g,
                     g.ro);
  hipLaunchKernelGGL(k_readout_scan, dim3(g.O), dim3(64), 0, s, g, g.ro);
  return hipGetLastError();
}

hipError_t bptt_forward_epilogue(const BpttArgs &a, const int32_t *labels, float *loss, hipStream_t s) {
  hipLaunchKernelGGL(k_loss, dim3(1), dim3(64), 0, s, a, labels, loss);
  return hipGetLastError();
}

hipError_t bptt_backward_prologue(const BpttArgs &a, const float *g_loss, hipStream_t s) {
  hipError_t e = hipSuccess;
  if (a.events) e = bptt_spike_masks(a, s);
  else gather_weights(a, s);
  if (a.seq_threads) {
    if (a.nnz_rec)
      hipLaunchKernelGGL(k_scatter_rows, dim3(blocks_for(a.nnz_rec, 256)), dim3(256), 0, s, a.w_rec, a.seq_pos, a.seq_w,
                         a.nnz_rec);
  } else {
    // the body is replayed from a graph, with copies of the weights
    if (e == hipSuccess)
      e = hipMemcpyAsync(a.w_out_c, a.w_out, (size_t)a.H * a.O * 4, hipMemcpyDeviceToDevice, s);
    if (a.S && a.nnz_rec)
      hipLaunchKernelGGL(k_scatter_pairs, dim3(blocks_for(a.nnz_rec, 256)), dim3(256), 0, s, a.w_rec, a.adj_pos,
                         a.adj_pair, a.nnz_rec);
    else if (e == hipSuccess && a.nnz_rec)
      e = hipMemcpyAsync(a.w_rec_c, a.w_rec, (size_t)a.nnz_rec * 4, hipMemcpyDeviceToDevice, s);
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_lam_u, dim3(a.O), dim3(64), 0, s, a, g_loss);
  return hipGetLastError();
}

// g: the plan's arguments with w_out = w_out_c and w_rec = w_rec_c
hipError_t bptt_backward_body(const BpttArgs &g, hipStream_t s) {
  if (g.seq_threads) {  // two kernels, launched without a graph
    hipLaunchKernelGGL(k_readout_adjoint_slice, dim3(blocks_for(g.H, kAdjointRows), g.T), dim3(256), 0, s, g, g.lamv);
    const dim3 grid(g.S == 8 ? 64u : g.B), block(g.seq_threads);
    if (g.seq_max <= 2) hipLaunchKernelGGL(k_adjoint_seq<8>, grid, block, 0, s, g);
    else if (g.seq_max <= 6) hipLaunchKernelGGL(k_adjoint_seq<24>, grid, block, 0, s, g);
    else hipLaunchKernelGGL(k_adjoint_seq<kSeqRegs>, grid, block, (size_t)g.seq_more_all * kWave * kSeqGroupBytes, s, g);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_fill, dim3(blocks_for((uint64_t)g.H * 64, 256)), dim3(256), 0, s, g.lam_carry,
                     (uint64_t)g.H * 64, 0.0f);
  // batch masks of the hidden trajectory for the sparse-weight gradients: in spiking
  // mode the forward pass wrote them (and flags[1] stayed clear); in smooth mode they are
  // taken here, and flag that the values are not binary
  if (g.smooth)
    hipLaunchKernelGGL(k_bits, dim3(blocks_for((uint64_t)g.T * g.H, 4)), dim3(256), 0, s, g.s, g.H, g.T, g.B,
                       g.sbits, g.flags + 1);
  // the readout part of every step's spike adjoint, into lamv (each adjoint step reads
  // its own entries, then overwrites them with lamV_t)
  if (g.S)
    hipLaunchKernelGGL(k_readout_adjoint_slice, dim3(blocks_for(g.H, kAdjointRows), g.T), dim3(256), 0, s, g, g.lamv);
  else
    hipLaunchKernelGGL(k_readout_adjoint, dim3(blocks_for((uint64_t)g.T * g.H, 4)), dim3(256), 0, s, g, g.lamv);
  const size_t slices = (size_t)g.S * g.H * 8;
  if (g.events) {
    // the forward pass kept the membranes of every step
    for (uint32_t t = g.T; t-- > 0;)
      hipLaunchKernelGGL(k_adjoint_slice, dim3(g.S * blocks_for(g.H, kAdjointRows)), dim3(1024), (size_t)g.H * 32, s, g,
                         g.sg + t * slices,
                         t + 1 < g.T ? g.lamv + (t + 1) * slices : g.lam_carry, g.lamv + t * slices);
    return hipGetLastError();
  }
  const dim3 grid(blocks_for(g.H, 4));
  const uint32_t n_seg = (g.T + g.K - 1) / g.K;
  for (int32_t seg = (int32_t)n_seg - 1; seg >= 0; --seg) {
    const uint32_t t0 = (uint32_t)seg * g.K, len = std::min(g.K, g.T - t0);
    // recompute the segment's membranes from the checkpoint before it and the stored
    // spikes (the forward pass's operations): all its currents at once, then the scan
    const float *vprev = seg ? g.vck + (size_t)(seg - 1) * g.H * 64 : nullptr;
    if (g.smooth)
      hipLaunchKernelGGL(k_seg_current_values, dim3(blocks_for((uint64_t)len * g.H, 4)), dim3(256), 0, s, g, t0,
                         len, g.vseg);
    else
      hipLaunchKernelGGL(k_seg_current, dim3(blocks_for((uint64_t)((len + kMaskSteps - 1) / kMaskSteps) * g.H, 4)),
                         dim3(256), 0, s, g, t0, len, g.vseg);
    hipLaunchKernelGGL(k_seg_scan, dim3(blocks_for((uint64_t)g.H * 64, 256)), dim3(256), 0, s, g, t0, len, vprev,
                       g.vseg);
    for (int32_t k = (int32_t)len - 1; k >= 0; --k) {
      const uint32_t t = t0 + (uint32_t)k;
      if (g.S) {
        hipLaunchKernelGGL(k_adjoint_slice, dim3(g.S * blocks_for(g.H, kAdjointRows)), dim3(1024), (size_t)g.H * 32, s, g,
                           g.vseg + (size_t)k * g.H * 64,
                           t + 1 < g.T ? g.lamv + (t + 1) * slices : g.lam_carry, g.lamv + t * slices);
        continue;
      }
      const float *lam_next = t + 1 < g.T ? g.lamv + (size_t)(t + 1) * g.H * 64 : g.lam_carry;
      hipLaunchKernelGGL(k_adjoint_step, grid, dim3(256), 0, s, g, t, g.vseg + (size_t)k * g.H * 64, lam_next,
                         g.lamv + (size_t)t * g.H * 64);
    }
  }
  return hipGetLastError();
}

// The dynamic LDS of the plan's kernels, once per plan.
hipError_t bptt_prepare(const BpttArgs &a) {
  auto allow = [](const void *k, size_t bytes) {
    return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  };
  hipError_t e = hipSuccess;
  if (a.S) e = allow(reinterpret_cast<const void *>(&k_adjoint_slice), kSliceMaxNeurons * 32u);
  if (e == hipSuccess && a.events) {
    e = allow(reinterpret_cast<const void *>(&k_hidden_seq<4>), kEventMaxNeurons * kSeqChunk * sizeof(float));
    if (e == hipSuccess) e = allow(reinterpret_cast<const void *>(&k_hidden_seq<2>), 1024u * kSeqChunk * sizeof(float));
    if (e == hipSuccess)
      e = allow(reinterpret_cast<const void *>(&k_adjoint_seq<kSeqRegs>), kSeqMaxMore * kWave * kSeqGroupBytes);
  }
  return e;
}

hipError_t bptt_fill_layouts(const BpttArgs &a, const BpttLayouts &lay, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_layouts, dim3(blocks_for(a.H, 4)), dim3(256), 0, s, a, lay);
  return hipGetLastError();
}

uint64_t bptt_lists(const BpttArgs &a) { return (uint64_t)(a.C + a.H) * blocks_for(a.T, kListChunk); }
uint32_t bptt_list_stride() { return kListStride; }

hipError_t bptt_trace_v(const BpttArgs &a, hipStream_t s) {
  const uint64_t n = (uint64_t)((a.T + a.K - 1) / a.K) * a.H * 64;
  hipLaunchKernelGGL(k_trace_v, dim3(blocks_for(n, 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

// the gradients, written to the caller's arrays
hipError_t bptt_backward_epilogue(const BpttArgs &a, hipStream_t s) {
  if (a.events)
    hipLaunchKernelGGL(k_grad_out_events, dim3(blocks_for((uint64_t)a.H * blocks_for(a.O, kOutBlock), 4)), dim3(256), 0, s,
                       a);
  else
    hipLaunchKernelGGL(k_grad_out, dim3(blocks_for((uint64_t)a.H * a.O, 4)), dim3(256), 0, s, a);
  if (a.events && a.nnz_in + a.nnz_rec) {
    const uint32_t n_lists = (a.C + a.H) * blocks_for(a.T, kListChunk);
    hipLaunchKernelGGL(k_event_lists, dim3(blocks_for(n_lists, 4)), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_grad_lists, dim3(blocks_for(a.H, 4 * kXcdCount) * 4 * kXcdCount), dim3(kGradBlock), 0, s, a);
  } else if (a.nnz_in + a.nnz_rec)
    hipLaunchKernelGGL(k_grad_edges, dim3(a.H), dim3(kGradBlock), (size_t)std::min(kGradChunk, a.T) * 64 * 4, s, a,
                       a.xbits, a.sbits, a.flags);
  return hipGetLastError();
}

}  // namespace snn
