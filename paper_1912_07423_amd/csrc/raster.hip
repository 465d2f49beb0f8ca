// raster.hip -- timestamped spike download (Sec. III-B): the set bits of a range of raster
// rows as (step, id) pairs, sorted by step and then by id.
//
// The rows' words, taken in step order, are cut into units of 64 x `iters` consecutive
// words, one wavefront each.  A count pass leaves every unit's number of spikes, one
// workgroup turns the counts into offsets, and an emit pass writes each unit's pairs from
// its offset on: lanes take consecutive words and every lane writes its word's bits in
// ascending order, so the pairs come out sorted.  The pairs go straight to pinned host
// memory, so that only spikes, not rows, cross the bus: 367 spikes of a 200,000-neuron
// step are 2.9 KB where its row is 25 KB.  Ranges of at most kSmallWords words take one
// launch of one workgroup instead of three.  Bound: the read of the rows (25 MB for 1,000
// such steps) and the host's copy out of the staging.  With every row copied to the host
// and scanned there, twice per download, 1,000 steps of 200,000 neurons (367,000 spikes)
// took 9.2 ms; they take 0.33 ms.
#include <algorithm>

#include "device_math.h"
#include "raster_units.h"
#include "snn_internal.h"

namespace snn {
namespace {

static_assert(kUnitLanes == kWave, "a unit is whole rounds of a wavefront");
constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kSmallBlock = 1024;
constexpr int kSmallWaves = kSmallBlock / kWave;

// Word x of the range (x < a.total_words): the range may wrap once around the ring.
__device__ __forceinline__ uint64_t raster_word(const RasterArgs &a, uint64_t x) {
  uint64_t at = a.first_word + x;
  if (at >= a.ring_words) at -= a.ring_words;
  return a.raster[at];
}

// Spikes of the words [lo, hi), by the whole wavefront.
__device__ __forceinline__ uint32_t count_words(const RasterArgs &a, uint64_t lo, uint64_t hi) {
  uint32_t c = 0;
#pragma unroll 4
  for (uint64_t x = lo + lane_id(); x < hi; x += kWave) c += (uint32_t)__popcll(raster_word(a, x));
  return wave_sum(c);
}

// Writes the pairs of the words [lo, hi) from position `at` on; positions outside
// [a.out_lo, a.out_lo + a.out_cap) are skipped.  Every lane of the wavefront runs every
// iteration (the scan needs them all).
__device__ __forceinline__ void emit_words(const RasterArgs &a, uint64_t lo, uint64_t hi, uint64_t at) {
  for (uint64_t base = lo; base < hi; base += kWave) {
    const uint64_t x = base + lane_id();
    uint64_t m = x < hi ? raster_word(a, x) : 0ull;
    const uint32_t c = (uint32_t)__popcll(m);
    const uint32_t incl = wave_inclusive_scan(c);
    if (m) {
      const uint64_t row = x / a.words;
      const uint32_t step = (uint32_t)(a.t_begin + row), id0 = (uint32_t)(x - row * a.words) * 64u;
      for (uint64_t p = at + (incl - c) - a.out_lo; m; ++p, m &= m - 1) {
        if (p < a.out_cap) {  // (a position below out_lo wraps to a large value)
          a.steps[p] = step;
          a.ids[p] = id0 + (uint32_t)__builtin_ctzll(m);
        }
      }
    }
    at += (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
  }
}

__global__ __launch_bounds__(kBlock) void k_raster_count(RasterArgs a) {
  const uint32_t unit = blockIdx.x * kWavesPerBlock + threadIdx.x / kWave;
  if (unit >= a.units) return;
  const uint64_t lo = (uint64_t)unit * a.unit_words, hi = std::min<uint64_t>(lo + a.unit_words, a.total_words);
  const uint32_t c = count_words(a, lo, hi);
  if (lane_id() == 0) a.offset[unit] = c;
}

// Counts to exclusive offsets in place (one workgroup), the total to *a.count.
__global__ __launch_bounds__(kSmallBlock) void k_raster_offsets(RasterArgs a) {
  __shared__ uint64_t wave_tot[kSmallWaves];
  const uint32_t w = threadIdx.x / kWave;
  uint64_t carry = 0;
  for (uint32_t base = 0; base < a.units; base += kSmallBlock) {
    const uint32_t u = base + threadIdx.x;
    const uint64_t c = u < a.units ? a.offset[u] : 0ull;
    const uint64_t incl = wave_inclusive_scan(c);
    if (lane_id() == kWave - 1) wave_tot[w] = incl;
    __syncthreads();
    uint64_t before = 0, all = 0;
#pragma unroll
    for (int v = 0; v < kSmallWaves; ++v) {
      before += (uint32_t)v < w ? wave_tot[v] : 0ull;
      all += wave_tot[v];
    }
    if (u < a.units) a.offset[u] = carry + before + incl - c;
    carry += all;
    __syncthreads();
  }
  if (threadIdx.x == 0) *a.count = carry;
}

__global__ __launch_bounds__(kBlock) void k_raster_emit(RasterArgs a) {
  const uint32_t unit = blockIdx.x * kWavesPerBlock + threadIdx.x / kWave;
  if (unit >= a.units) return;
  const uint64_t lo = (uint64_t)unit * a.unit_words, hi = std::min<uint64_t>(lo + a.unit_words, a.total_words);
  emit_words(a, lo, hi, a.offset[unit]);
}

// The three passes of a short range in one workgroup: a wavefront per contiguous sixteenth.
__global__ __launch_bounds__(kSmallBlock) void k_raster_small(RasterArgs a) {
  __shared__ uint32_t tot[kSmallWaves];
  const uint32_t w = threadIdx.x / kWave;
  const uint64_t share = (a.total_words + kSmallBlock - 1) / kSmallBlock * kWave;
  const uint64_t lo = std::min<uint64_t>(w * share, a.total_words), hi = std::min<uint64_t>(lo + share, a.total_words);
  const uint32_t c = count_words(a, lo, hi);
  if (lane_id() == 0) tot[w] = c;
  __syncthreads();
  uint64_t before = 0, all = 0;
#pragma unroll
  for (int v = 0; v < kSmallWaves; ++v) {
    before += (uint32_t)v < w ? tot[v] : 0u;
    all += tot[v];
  }
  if (threadIdx.x == 0) *a.count = all;
  emit_words(a, lo, hi, before);
}

// One workgroup reads 16 words per lane of a range of this size, about what the two further
// launches of the general form cost (2.5 us each).
constexpr uint64_t kSmallWords = 16384;

}  // namespace

// Counts the range's spikes into *a.count and, with a.out_cap > 0, writes the pairs.  The
// range is not empty.
hipError_t launch_raster_pairs(RasterArgs a, hipStream_t s) {
  if (a.total_words <= kSmallWords) {
    k_raster_small<<<1, kSmallBlock, 0, s>>>(a);
    return hipGetLastError();
  }
  const uint64_t units = raster_units(a.total_words, &a.unit_words);
  if (units > a.scratch) return hipErrorInvalidValue;
  a.units = (uint32_t)units;
  const uint32_t grid = (a.units + kWavesPerBlock - 1) / kWavesPerBlock;
  k_raster_count<<<grid, kBlock, 0, s>>>(a);
  k_raster_offsets<<<1, kSmallBlock, 0, s>>>(a);
  if (a.out_cap) k_raster_emit<<<grid, kBlock, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace snn
