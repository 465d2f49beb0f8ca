// snn_internal.h -- library-private types shared by the host runtime and kernels.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "../../include/snn.h"

namespace snn {

constexpr uint32_t kTableCap = 256;

// Many workgroups update the same counters at the same moment; same-line atomics
// from a burst of workgroups serialise, so every shared counter gets its own
// 256-byte line and the hot ones are split into independent parts.
constexpr uint32_t kQlenStride = 64;    // uint32 per counter line
constexpr uint32_t kLineU64 = 32;       // uint64 per 256-byte line
constexpr uint32_t kQueueGroups = 8;    // sub-queues of a step's spike queue
constexpr uint32_t kCounterParts = 64;  // partial sums of the event/spike/touch counters
constexpr uint32_t kUpdateBlock = 256;  // neurons per update workgroup
constexpr uint32_t kGuideBits = 12;     // drive guide table: buckets on the top bits of r
constexpr uint32_t kGuideBuckets = 1u << kGuideBits;

// Device-resident control block.  `t` is the first step of the next update launch;
// the update launch copies it to `t_deliver` and the delivery launch that closes the
// window advances `t`, so every kernel finds its step on the device and a captured
// HIP graph replays correctly.
struct Ctl {
  uint64_t t;
  uint64_t t_deliver;
  uint64_t lazy_overrun;  // rows found with more pending steps than the history holds
  uint64_t pad[kLineU64 - 3];
  uint64_t events[kCounterParts * kLineU64];   // part p at [p * kLineU64]
  uint64_t spikes[kCounterParts * kLineU64];
  uint64_t touches[kCounterParts * kLineU64];
};

// A step's spike queue is kQueueGroups sub-queues of group_cap entries each; update
// workgroup b appends to sub-queue b % kQueueGroups.  Counter of (slot, group) at
// qlen[(slot * kQueueGroups + group) * kQlenStride].
struct QueueRef {
  int32_t *ids;       // [slots][stride]
  uint32_t *qlen;
  uint32_t stride;    // kQueueGroups * group_cap
  uint32_t group_cap;
};

// One projection as the device generators see it (per source population, sorted by
// first target population).
struct GenProj {
  uint32_t kind;     // SNN_PROJ_*
  uint32_t k;        // out-degree (fixed)
  uint32_t first_pop;  // first target population (stream id of the fixed generator)
  uint32_t off;      // first target id
  uint32_t size;     // number of target ids
  uint32_t self_in;  // sources of this projection lie inside the target range
  uint32_t plastic;
  int32_t w_q16;
  float w_f32;
  uint32_t pad;
  uint64_t thr;      // ER: edge iff word < thr
  uint64_t spare;    // fixed: candidates - k
};

struct GenArgs {
  const GenProj *proj;      // [n_proj] sorted by (source population, first target)
  const uint32_t *pop_off;  // [n_pops + 1]
  const uint32_t *pop_proj; // [n_pops + 1] projection range of each source population
  uint32_t n_pops, n;
  uint32_t key0, key1;
};

// Lazy plasticity (Sec. III-A.1, Table I "bitmasks", "ages", "expirations").  Row i's
// potentiation events of the steps [age_i, t] are pending: they wait in the targets'
// spike histories and are applied when the row transmits or, at the latest, when the
// oldest pending step is about to leave the kLazyHistory-step history.
constexpr uint32_t kLazyHistory = 64;  // steps of spike history per neuron (one uint64)
struct LazyRef {
  uint64_t *hist;         // [n] bit k: the neuron spiked at step t - k (t the last update)
  uint32_t *age;          // [n] first pending step of the row, mod 2^32
  float *x_age;           // [n] the row's presynaptic trace at its age step
  const uint32_t *plast_len;  // [n] plastic synapses of each row (0: no age kept)
  QueueRef exq;           // 2 slots: the expiring rows of step t in slot t mod 2, laid out
                          // as a spike queue (kQueueGroups sub-queues)
  uint32_t delay;
};

struct UpdateArgs {
  float *v;
  int32_t *ref;
  int32_t *input;     // [n_inbuf][n]
  float *x_pre, *x_post;
  QueueRef q;
  uint64_t *raster;   // [raster_cap][words]
  const uint32_t *table32;  // drive thresholds below 2^32
  const uint16_t *guide;    // [kGuideBuckets]: count at the bucket's low end | high end << 8
  Ctl *ctl;
  uint32_t n, slots, n_inbuf, raster_cap, words, table_len;
  uint32_t key0, key1;
  float alpha, v_inf, v_th, v_reset, beta_plus, beta_minus;
  int32_t ref_steps, w_ext_q16;
  uint32_t zero_input, plastic;
  // lazy plasticity (one step per launch): spike history, ages and the expiring-row
  // queue, all null otherwise
  LazyRef lazy;
};

struct DeliverArgs {
  const uint64_t *row_ptr;
  const int32_t *col;
  const int32_t *w_q16;   // static networks with a weight per synapse
  const float *w_f32;     // plastic networks
  const int32_t *w_src;   // static networks with one weight per source population:
                          // Q16 weight of every synapse of source i (no w_q16)
  QueueRef q;
  int32_t *input;
  const uint16_t *col16;  // tiled delivery: low 16 bits of every target, [nnz] padded to
                          // whole 16-byte groups
  const void *tile_off;   // [n][tiles + 1] tile boundaries of each row, relative to the
                          // row's start: uint16 when off16, else uint32
  Ctl *ctl;
  uint32_t n, slots, n_inbuf, delay, window_max;
  uint32_t tiles, tile_size;
  uint32_t row_groups;    // 16-byte groups of targets of a mean row (tiled delivery)
  uint32_t off16;
  uint32_t advance;       // this launch closes the window: advance the step counter
  float *x_pre, *x_post;  // eager STDP: here x_pre += 1 for S_{t-d}, x_post += 1 for S_t (else null)
};

// The lazy plasticity kernel of one step t: rows of S_{t-d+1} transmit (pending
// potentiation applied, then delivered with the current weights), expiring rows are
// brought current, and the postsynaptic traces of S_t are incremented.
struct LazyArgs {
  const uint64_t *row_ptr;
  const int32_t *col;
  float *w_f32;
  const uint32_t *plast_rel;
  float *x_pre, *x_post;
  QueueRef q;
  int32_t *input;
  LazyRef lazy;
  Ctl *ctl;
  uint32_t n, slots, delay;
  float a_plus, w_max, beta_plus;
};

struct StdpArgs {
  const uint64_t *row_ptr;
  const int32_t *col;
  float *w_f32;
  const uint32_t *plast_rel, *plast_len;
  const uint64_t *in_ptr;
  const int32_t *in_src;
  const uint32_t *in_edge;
  float *x_pre, *x_post;
  QueueRef q;
  Ctl *ctl;
  const uint64_t *raster;  // [raster_cap][words] spike bits (the fused pass tests S_t, S_{t-d})
  uint32_t raster_cap, words;
  uint32_t n, slots, delay;
  float a_plus, a_minus, w_max;
};

// Windows of an eagerly plastic network (plastic.hip): a workgroup per range of targets.
constexpr uint32_t kPlasticBlock = 512;  // its lanes, and the most targets of a range
constexpr uint32_t kPlasticAhead = 8;    // sub-rows of a lane group in flight
constexpr uint32_t kPlasticRows = 2048;  // most arriving rows of a window that are laid out
constexpr uint32_t kPlasticSteps = 16;   // most steps of a window (its arrivals are one 32-bit mask)
// One arriving neuron's synapses on the range: [lo, lo + len), those from p0 to p1 (offsets
// from lo) plastic, and its presynaptic trace (the value at the window's start, and bit m: it
// arrives at step m of the window).  A row has at most one synapse per target (projections do
// not overlap), so len <= kPlasticBlock.
struct SubRow {
  uint32_t lo, dims;
  uint2 trace;
  __host__ __device__ uint32_t len() const { return dims & 1023u; }
  __host__ __device__ uint32_t p0() const { return (dims >> 10) & 1023u; }
  __host__ __device__ uint32_t p1() const { return dims >> 20; }
  // the latest arrival before step m (0: none), and whether there are several
  __host__ __device__ uint32_t from(uint32_t m) const {
    const uint32_t before = trace.y & ((1u << m) - 1u);
    return before ? 31u - (uint32_t)__builtin_clz(before) : 0u;
  }
  __host__ __device__ bool again() const { return (trace.y & (trace.y - 1u)) != 0; }
};
static_assert(kPlasticBlock < 1024 && kPlasticSteps < 32, "fields of SubRow");
struct PlasticArgs {
  const uint64_t *row_ptr;
  const int32_t *col;
  float *w_f32;
  const uint32_t *plast_rel, *plast_len;
  const uint64_t *in_ptr;
  const int32_t *in_src;
  const uint32_t *in_edge;
  const void *off;        // [n][ranges + 1] range boundaries of each row: uint16 when off16
  // of this window at [parity], of the window before at [parity ^ 1]:
  uint2 *trace[2];        // [n] presynaptic trace at the window's start, arrivals in its steps
  uint4 *ltp[2];          // [n] its spiking neurons: first in-edge, in-edges, spikes
  uint32_t *ltp_len[2];
  uint32_t parity;
  uint32_t first, last;   // window of the run
  int32_t *list;          // [list_slots][n] spikes of the latest steps
  uint32_t *list_len;     // [list_slots] on lines of their own
  uint32_t list_slots;
  uint32_t *arriving;     // [kPlasticSteps + 1] rows of the window's lists
  SubRow *row_head;       // [ranges][row_cap] arriving sub-rows,
  uint16_t *row_tgt;      // [ranges][row_cap][2^lanes_shift] their targets in the range
  uint32_t row_cap;
  uint32_t ltp_blocks, row_blocks;  // workgroups of the prepare launch
  float *v;
  int32_t *ref;
  int32_t *input;         // [n]
  float *x_pre, *x_post;
  QueueRef q;
  uint64_t *raster;
  const uint32_t *table32;
  const uint16_t *guide;
  Ctl *ctl;
  uint32_t n, slots, raster_cap, words, table_len, delay;
  uint32_t range, ranges, off16;
  uint32_t lanes_shift;   // log2 of the lanes that share one sub-row
  uint32_t key0, key1;
  float alpha, v_inf, v_th, v_reset, beta_plus, beta_minus;
  int32_t ref_steps, w_ext_q16;
  float a_plus, a_minus, w_max;
};
// The lists of the last `delay` steps, from the raster.
hipError_t launch_plastic_import(const PlasticArgs &a, hipStream_t s);
// steps <= min(delay - 1, kPlasticSteps) steps from ctl->t on.
hipError_t launch_plastic_window(const PlasticArgs &a, uint32_t steps, hipStream_t s);
// After the last window of a run (a as for a window that followed): the potentiation it
// left, and the FIFO ring.
hipError_t launch_plastic_export(const PlasticArgs &a, hipStream_t s);

// One network of a batch as the persistent batch kernel sees it: pointers into the
// network's own buffers (state layout identical to the single-network pipeline) and
// its derived constants.
struct BatchNet {
  const uint64_t *row_ptr;
  const int32_t *col, *w_q16;
  const int32_t *w_src;      // one weight per source neuron (then w_q16 is null)
  float *v;
  int32_t *ref;
  int32_t *input;            // [delay][n] Q16 accumulators, slot t mod delay
  int32_t *queue;            // [slots][queue_stride] the FIFO ring of spike queues
  uint32_t *qlen;            // its counters (written with kBatchQueues)
  uint64_t *raster;          // [raster_cap][words]
  const uint32_t *table32;   // drive thresholds below 2^32
  Ctl *ctl;
  uint32_t n, words, delay, raster_cap;
  uint32_t slots, queue_stride, group_cap, window;  // of the FIFO ring
  uint32_t below;            // number of drive thresholds below 2^32 (0: no drive)
  uint32_t lanes_shift;      // log2 of the lanes that share one spike's row
  uint32_t key0, key1;
  float alpha, v_inf, v_th, v_reset;
  int32_t ref_steps, w_ext_q16;
};
constexpr uint32_t kBatchCommit = 1u;       // write state, counters and t back
constexpr uint32_t kBatchWriteRaster = 2u;  // write the raster rows
constexpr uint32_t kBatchDrive = 4u;        // some member has a Poisson drive
constexpr uint32_t kBatchQueues = 8u;      // leave the FIFO ring as the step pipeline does
constexpr uint32_t kBatchStaticLds = 64u;   // bound on the kernels' static LDS
constexpr uint32_t kBatchQueueMax = 512u;   // queue entries in LDS (12 bytes each)
constexpr uint32_t kSoloMaxNeurons = 40960u;
// Dynamic LDS of a persistent launch in 4-byte words: a network's accumulators and drive
// thresholds, q_cap queue entries of three words, and, for the networks whose n + 1 row offsets fit behind
// them, those.
struct LdsPlan {
  uint32_t words, q_cap;
};
bool batch_variant_supported(uint32_t block, uint32_t per);
uint32_t batch_per_lane(uint32_t block, uint32_t n_max);  // 0: n_max too large for block
hipError_t launch_batch(const BatchNet *nets, const uint32_t *order, uint32_t n_nets, uint32_t steps,
                        uint32_t block, uint32_t per, uint32_t flags, LdsPlan lds, hipStream_t s);
// One network of at most kSoloMaxNeurons neurons without drive by itself (one workgroup).
hipError_t launch_solo(const BatchNet &d, uint32_t steps, uint32_t flags, LdsPlan lds, hipStream_t s);

// Surrogate-gradient BPTT plan as its kernels see it (bptt.hip).  Batch <= 64: lane b
// of a wavefront is batch element b; sizes are B batch, T steps, C inputs, H hidden,
// O readouts, K steps per checkpoint segment (<= 32).
// Limits of the ELL form of the hidden steps: rows of at most 256 in-edges (four lane
// loads), and at most 8,192 hidden neurons (their 64 KiB of spike masks in LDS).
constexpr uint32_t kEllMaxWidth = 256;
constexpr uint32_t kEllMaxNeurons = 8192;
// The sliced membrane adjoint: a slice of all neurons (32 bytes each) is staged in LDS, and
// the synapses are held as padded rows of at most kSliceMaxPairs entries in all.
constexpr uint32_t kSliceMaxNeurons = 4096;
constexpr int kAdjointRows = 32;  // neurons per workgroup of the sliced kernels
// The event-driven forward pass holds the weights as dense rows: at most 2,048 hidden neurons
// (16 MB of recurrent weights; a presynaptic spike costs a whole row of them) and 64 MB of
// input weights.
constexpr uint32_t kEventMaxNeurons = 2048;
constexpr uint64_t kEventMaxInput = 1ull << 24;
// The membrane adjoint of one batch element in one workgroup: at most kSeqMaxNeurons neurons;
// kSeqRegs synapses of a lane in registers, the others in LDS, in groups of four (24 bytes)
// per lane, at most kSeqMaxMore groups per wavefront in all (150 KB).
constexpr uint32_t kSeqMaxNeurons = 1024;
constexpr int kSeqRegs = 48;
constexpr uint32_t kSeqGroupBytes = 24;
constexpr uint32_t kSeqMaxMore = 98;
constexpr uint64_t kSliceMaxPairs = 1ull << 26;
constexpr uint32_t kActSamples = 1024;  // words that a pass's activity is estimated from
struct BpttArgs {
  uint32_t B, T, C, H, O, K;
  uint32_t events;             // event-driven forward pass (spiking mode); then also:
  uint32_t Hp, nw, col_w;      // columns of a dense row (multiple of 256), words of 64 neurons,
                               // longest column of W_rec
  float *dense_in, *dense_rec; // [C][Hp], [H][Hp]
  uint2 *col_pair;             // [col_w][Hp] (source, weight) in ascending source order
  const uint32_t *in_pos, *rec_pos, *col_pos;  // place of each CSR edge in them
  float *vall;                 // [T][B][Hp] input currents, then membranes of every step
  float *sg;                   // [T][S][H][8] surrogate derivatives (backward pass)
  uint16_t *lists;             // event lists of every source and chunk of steps
  uint32_t *list_len;          // their lengths
  uint64_t *spk;               // [B][T][nw] spikes of every step
  uint32_t seq_threads;        // lanes of a one-workgroup membrane adjoint (0: steps launched)
  uint32_t seq_p, seq_max;     // lanes per neuron, groups of four synapses of the longest wavefront
  const uint32_t *seq_row;     // [seq_threads] neuron of each lane (0xFFFFFFFF: none)
  const uint32_t *seq_groups;  // [16] groups of four synapses of each wavefront's lanes
  const uint32_t *seq_more;    // [16] first LDS group of each wavefront
  uint32_t seq_more_all;       // LDS groups of all wavefronts
  const uint16_t *seq_col;     // [seq_max][seq_threads][4] LDS offsets of the targets
  float *seq_w;                // [seq_max][seq_threads][4] weights
  const uint32_t *seq_pos;     // [nnz_rec] place of each CSR edge in seq_w
  uint32_t S;                  // slices of 8 batch elements of the membrane adjoint (0: not sliced)
  uint32_t adj_w;              // width of its padded rows of W_rec, a multiple of 16
  uint2 *adj_pair;             // [H][adj_w] (target, weight); padding (0, 0)
  const uint32_t *adj_pos;     // [nnz_rec] place of each CSR edge
  const uint32_t *adj_len;     // [H] row lengths
  float beta, beta_out, theta, slope;
  uint32_t smooth, detach_reset;
  uint64_t nnz_in, nnz_rec;
  const uint64_t *in_t_ptr;    // W_in transposed: in-edges of each hidden neuron,
  const int32_t *in_t_src;     //   sources ascending, with their CSR edge index
  const uint32_t *in_t_edge;
  const uint64_t *rec_t_ptr;   // W_rec transposed, likewise
  const int32_t *rec_t_src;
  const uint32_t *rec_t_edge;
  const uint64_t *rec_ptr;     // W_rec forward rows
  const int32_t *rec_col;
  const float *w_in, *w_rec, *w_out;  // caller's weights: CSR order, CSR order, [H][O]
  float *g_w_in, *g_w_rec, *g_w_out;
  float *w_in_t, *w_rec_t;     // weights gathered into transposed (per-target) order
  float *w_out_c, *w_rec_c;    // the plan's copies of w_out and of w_rec in CSR order
  float *iin;                  // [T][H][64] input-projection current of every step
  uint64_t *xbits, *sbits;     // batch masks of the input and hidden spikes: [C][T], [H][T]
  uint64_t *sbits_t;           // the hidden spike masks again, step-major: [T][H]
  uint32_t ell_w;              // width of the ELL copy of W_rec's in-edges (0: none)
  const int32_t *ell_src;      // [H][ell_w] sources, ascending, then 0-padding
  const uint32_t *ell_edge;    // [H][ell_w] CSR edge index (padding: 0xFFFFFFFF)
  const uint32_t *ell_len;     // [H] in-degree
  float *ell_wt;               // [H][ell_w] weights gathered into that order (padding: 0)
  uint32_t *flags;             // [4]: a value of x / s is neither 0 nor 1 (masks not used); event-driven
                               // form: a readout weight / adjoint is not finite (no term is left out)
  float *xt, *s, *vck, *vtmp, *vseg, *ro, *lamu, *lamv, *lam_carry, *m, *dm;
  int32_t *tmax;
  uint32_t *act_out;           // [3] set bits of kActSamples words of xbits and of spk, flags[0]: pinned
                               // host memory
};
// Forward and backward passes in three parts each: prologue and epilogue touch the
// caller's arrays, the body only the plan's buffers (capturable once per plan).  The body
// takes the plan's arguments with w_out (and, backward, w_rec) pointing at the plan's
// copies w_out_c / w_rec_c, which the prologue fills.
hipError_t bptt_prepare(const BpttArgs &a);
// The plan's index arrays that follow from the CSR forms (null: not used); col_pair and adj_pair get
// their sources and targets too.
struct BpttLayouts {
  uint32_t *in_pos, *rec_pos, *col_pos;  // event-driven form
  uint32_t *adj_pos, *adj_len;           // sliced adjoint
  int32_t *ell_src;                      // padded in-edges
  uint32_t *ell_edge, *ell_len;
};
hipError_t bptt_fill_layouts(const BpttArgs &a, const BpttLayouts &lay, hipStream_t s);
hipError_t bptt_spike_masks(const BpttArgs &a, hipStream_t s);
uint64_t bptt_lists(const BpttArgs &a);  // number of event lists, entries held for each
uint32_t bptt_list_stride();
hipError_t bptt_trace_v(const BpttArgs &a, hipStream_t s);  // fills vck (event-driven plans)
// busy (event-driven plans): the input currents by masks and the hidden steps by launches
// (bptt_forward_body), for passes whose activity makes that the faster way; else bptt_hidden_seq.
// Either is followed by bptt_readout_events, and the results are the same bit for bit.
hipError_t bptt_forward_prologue(const BpttArgs &a, const float *x, bool busy, hipStream_t s);
hipError_t bptt_hidden_seq(const BpttArgs &a, hipStream_t s);
hipError_t bptt_readout_events(const BpttArgs &a, bool busy, hipStream_t s);
hipError_t bptt_forward_body(const BpttArgs &g, hipStream_t s);
hipError_t bptt_forward_epilogue(const BpttArgs &a, const int32_t *labels, float *loss, hipStream_t s);
hipError_t bptt_backward_prologue(const BpttArgs &a, const float *g_loss, hipStream_t s);
hipError_t bptt_backward_body(const BpttArgs &g, hipStream_t s);
hipError_t bptt_backward_epilogue(const BpttArgs &a, hipStream_t s);

// Optional timing events of one launch.  When set, the kernel is launched with
// hipExtLaunchKernel, which stamps `start` and `stop` with the dispatch's own begin and
// end (no marker packet is placed between launches); launches that span two kernels
// stamp the first one's begin and the last one's end.
struct LaunchEvents {
  hipEvent_t start = nullptr, stop = nullptr;
  bool on() const { return start != nullptr || stop != nullptr; }
};

// Spike download (raster.hip): the (step, id) pairs of a range of raster rows.
struct RasterArgs {
  const uint64_t *raster;
  uint64_t ring_words;    // raster_cap * words
  uint64_t first_word;    // ring position of the range's first word
  uint64_t total_words;   // rows * words
  uint64_t t_begin;
  uint64_t unit_words;    // words per unit (set by the launcher)
  uint64_t *offset;       // [scratch] counts, then offsets of the units
  uint64_t scratch;       // entries of offset: at least the range's units (raster_units.h)
  uint64_t *count;        // host-visible: spikes in the range
  uint32_t *steps, *ids;  // host-visible: pairs [out_lo, out_lo + out_cap)
  uint64_t out_lo, out_cap;
  uint32_t words, units;
};
hipError_t launch_raster_pairs(RasterArgs a, hipStream_t s);

// kernel launchers (step.hip / generate.hip)
hipError_t launch_update(const UpdateArgs &a, uint32_t steps, hipStream_t s, const LaunchEvents &ev = {});
hipError_t launch_deliver_atomic(const DeliverArgs &a, uint32_t steps, uint32_t grid,
                                 hipStream_t s, const LaunchEvents &ev = {});
hipError_t launch_deliver_tiled(const DeliverArgs &a, uint32_t steps, uint32_t block,
                                uint32_t grid, hipStream_t s, const LaunchEvents &ev = {});
constexpr uint32_t kTileGroupMax = 32;  // base tiles one tiled-delivery workgroup may own
hipError_t prepare_deliver_tiled(uint32_t block, size_t *max_dynamic_lds);
hipError_t launch_stdp_ltd(const StdpArgs &a, uint32_t grid, hipStream_t s, const LaunchEvents &ev = {});
hipError_t launch_stdp_fused(const StdpArgs &a, uint32_t grid, hipStream_t s, const LaunchEvents &ev = {});
hipError_t launch_lazy(const LazyArgs &a, uint32_t grid, hipStream_t s, const LaunchEvents &ev = {});
// Brings every plastic row current at step boundary t (pending potentiation applied,
// age t, trace at age rebuilt from x_pre and the arrivals of step t).
hipError_t launch_lazy_flush(const LazyArgs &a, uint64_t t, uint32_t grid, hipStream_t s);
// One window's queues staged from a caller's spike list (k_stage_window): step w's
// ids are ids[off[w] .. off[w+1]), or dealt round-robin over the steps when
// round_robin is set (off then still holds each step's count as a prefix).
struct StageArgs {
  QueueRef q;             // `steps` slots
  Ctl *ctl;
  int32_t *input;         // n_input accumulators, cleared
  const int32_t *ids;
  uint64_t n_input;
  uint64_t t_deliver;
  uint32_t n_ids, steps, round_robin;
  uint32_t off[65];       // steps <= 64
};
hipError_t launch_stage_window(const StageArgs &a, hipStream_t s);
hipError_t launch_row_lengths(const GenArgs &g, uint32_t *len, uint32_t *plast_rel,
                              uint32_t *plast_len, hipStream_t s);
// Indexes of the tiled delivery, written by the fill as well if col16 is not null (then every
// population has at most one projection, of fixed out-degree).
struct RowIndex {
  uint16_t *col16;     // [count]
  void *tile_off;      // [n][tiles + 1], uint16 if off16
  uint64_t nnz, count;
  uint32_t tiles, tile_size;
  bool off16;
  uint32_t inv32;      // set by the launcher
};
// all_fixed: every projection is fixed out-degree (no ER rows), which allows one
// workgroup per row for long rows.
hipError_t launch_fill_rows(const GenArgs &g, uint32_t max_fixed_k, bool all_fixed, const uint64_t *row_ptr,
                            int32_t *col, int32_t *w_q16, float *w_f32, RowIndex index, hipStream_t s);
hipError_t launch_spacing_gaps(const uint32_t *words, uint64_t n, uint32_t *gaps, hipStream_t s);
hipError_t launch_scan_u32_to_u64(const uint32_t *in, uint64_t *out, uint32_t n,
                                  uint64_t *block_sums, hipStream_t s);
size_t scan_scratch_elems(uint32_t n);
hipError_t launch_count_in_edges(const uint64_t *row_ptr, const int32_t *col,
                                 const uint32_t *plast_rel, const uint32_t *plast_len,
                                 uint32_t n, uint32_t *count, hipStream_t s);
hipError_t launch_fill_in_edges(const uint64_t *row_ptr, const int32_t *col,
                                const uint32_t *plast_rel, const uint32_t *plast_len,
                                uint32_t n, uint64_t *cursor, int32_t *in_src,
                                uint32_t *in_edge, hipStream_t s);
hipError_t launch_tile_index(const uint64_t *row_ptr, const int32_t *col, uint32_t n, uint64_t nnz,
                             uint64_t count, uint32_t tiles, uint32_t tile_size, uint16_t *col16,
                             void *tile_off, bool off16, hipStream_t s);
hipError_t launch_init_neurons(float *v, int32_t *ref, uint32_t n, uint32_t key0, uint32_t key1,
                               float lo, float span, hipStream_t s);

}  // namespace snn

// The network object behind the opaque handle.
struct snn_network {
  // description
  std::vector<snn_population> pops;
  std::vector<snn_projection> proj;
  std::vector<uint32_t> pop_off;
  snn_params prm;
  // setup timing (host wall time of the build; device time of its generation phases)
  double build_ms = 0;
  float gen_rows_ms = 0, gen_fill_ms = 0, index_ms = 0;
  uint32_t key0 = 0, key1 = 0;

  // sizes and schedule
  uint32_t n = 0, delay = 1, slots = 2, n_inbuf = 1, window = 1;
  uint32_t delivery = SNN_DELIVERY_ATOMIC, tiles = 1, tile_size = 1, block = 512, grid = 512;
  uint32_t raster_cap = 1024, words = 1;
  bool plastic = false;
  bool lazy = false;  // plastic, with SNN_PLASTICITY_LAZY
  uint64_t nnz = 0, nnz_alloc = 0;

  // derived constants
  float alpha = 0, v_inf = 0, v_th = 0, v_reset = 0;
  float beta_plus = 0, beta_minus = 0, a_plus = 0, a_minus = 0, w_max = 0;
  int32_t ref_steps = 0, w_ext_q16 = 0;
  uint64_t table[snn::kTableCap] = {};
  uint32_t table_len = 0;

  // device memory
  uint64_t *row_ptr = nullptr;
  int32_t *col = nullptr, *w_q16 = nullptr;
  float *w_f32 = nullptr;
  int32_t *w_src = nullptr;             // per-source weights (Table I layout)
  std::vector<int32_t> w_src_host;
  uint32_t *plast_rel = nullptr, *plast_len = nullptr;
  uint64_t *in_ptr = nullptr;
  int32_t *in_src = nullptr;
  uint32_t *in_edge = nullptr;
  void *tile_off = nullptr;
  uint16_t *col16 = nullptr;   // low 16 bits of every target (tiled delivery)
  bool tile_off16 = false;    // tile boundaries stored as uint16 (every row < 65,536 synapses)
  uint64_t row_len_bound = 0; // upper bound on a row's length, from the projections
  float *v = nullptr, *x_pre = nullptr, *x_post = nullptr;
  int32_t *ref = nullptr, *input = nullptr, *queue = nullptr;
  uint32_t *qlen = nullptr;
  uint32_t queue_stride = 0, group_cap = 0;  // entries per queue slot / per sub-queue
  uint64_t *raster = nullptr;
  uint64_t *raster_offset = nullptr;  // scratch of the spike download, its entries
  uint64_t raster_scratch = 0;
  uint32_t *d_table32 = nullptr;
  uint16_t *d_guide = nullptr;
  snn::Ctl *ctl = nullptr;
  // eager plasticity: windows of steps in one launch (plastic.hip)
  bool windows = false;       // snn_run takes them
  uint64_t windows_from = 0;  // from this step on (the raster then holds every pending queue)
  void *range_off = nullptr;  // range boundaries of every row
  uint2 *trace = nullptr;     // [2][n]
  uint4 *ltp = nullptr;       // [2][n]
  int32_t *spike_list = nullptr;
  uint32_t *spike_list_len = nullptr;  // [list_slots + 3], the last three for ltp and arriving
  snn::SubRow *row_head = nullptr;
  uint16_t *row_tgt = nullptr;
  uint32_t list_slots = 0, row_cap = 0, row_shift = 0;
  uint32_t range = 0, ranges = 0;
  // lazy plasticity: per-neuron spike history, row ages and traces at age, expiring rows
  uint64_t *hist = nullptr;
  uint32_t *age = nullptr;
  float *x_age = nullptr;
  int32_t *exq = nullptr;
  uint32_t *exq_len = nullptr;

  // bookkeeping
  struct Alloc {
    void *p;
    size_t bytes;
  };
  std::vector<Alloc> allocs;
  snn_allocator alloc{};
  bool has_alloc = false;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  int device = 0;
  uint32_t cu_count = 256;
  uint64_t t_host = 0;  // steps issued (mirror of the device counter)
  snn_batch *owner = nullptr;  // set for the members of a batch
  uint64_t device_bytes = 0;

  bool delivery_chosen = false;  // by the caller, with the parameters or snn_set_delivery
  bool solo = false;         // snn_run may step it by the persistent one-workgroup kernel
  double spikes_per_step = -1.0;  // of its latest steps, where the route depends on it (< 0: not known)
  uint64_t rate_at = 0;           // the step at which that was found
  uint64_t rate_gap = 64;         // steps after which it is counted again
  double noted_spikes = 0.0;      // of downloads since then, and their steps
  uint64_t noted_steps = 0;
  uint32_t lds_limit = 0;    // largest workgroup LDS

  // graph of a fixed chunk of windows
  hipGraphExec_t graph = nullptr;
  uint32_t graph_steps = 0;

  // profiling: hipEvent pairs around launches, resolved at the next readout
  struct ProfRecord {
    int kind;  // 0 update, 1 deliver, 2 stdp
    hipEvent_t a, b;
  };
  bool profiling = false;
  snn_profile prof{};
  std::vector<ProfRecord> prof_pending;
  std::vector<hipEvent_t> event_pool;
};
