// raster_units.h -- how the spike download cuts a range of raster words into units.
#pragma once
#include <algorithm>
#include <cstdint>

namespace snn {

// Units of at least kMinUnitWords words, and few enough that one workgroup scans their
// counts in eight rounds.
constexpr uint64_t kMaxRasterUnits = 8192;
constexpr uint64_t kUnitLanes = 64;  // a unit's length is a multiple of a wavefront's lanes
constexpr uint64_t kMinUnitWords = 8 * kUnitLanes;

// Units of a range of `words` words, and their length.  The number does not grow steadily
// with the range: past kMaxRasterUnits of the shortest units their length goes up in steps, and
// the number falls back at every step.
inline uint64_t raster_units(uint64_t words, uint64_t *unit_words) {
  const uint64_t most = kMaxRasterUnits * kUnitLanes;
  const uint64_t unit = std::max(kMinUnitWords, (words + most - 1) / most * kUnitLanes);
  if (unit_words) *unit_words = unit;
  return (words + unit - 1) / unit;
}

// Entries of the offsets scratch of a ring of `ring_words` words: the most units that any range
// of up to that many words is cut into.
inline uint64_t raster_scratch(uint64_t ring_words) {
  return std::min(kMaxRasterUnits, (ring_words + kMinUnitWords - 1) / kMinUnitWords);
}

}  // namespace snn
