"""The offsets scratch of the spike download holds the units of every range that its ring can
be asked for.  The unit count falls back at every multiple of 524,288 words past 4,194,304, so
the whole ring is not the range with the most units: every range length is gone through by the
sizing functions themselves, compiled from their header with g++."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1912_07423_amd", "csrc")

PROGRAM = r"""
#include "raster_units.h"
#include <cstdio>
int main() {
  // most = units of the worst range up to `words`: a ring of `words` words needs that many
  unsigned long long most = 0, over = 0;
  for (unsigned long long words = 1; words <= (1ull << 26); ++words) {
    uint64_t unit = 0;
    const unsigned long long units = snn::raster_units(words, &unit);
    if (units > most) most = units;
    if (unit % 64 || units * unit < words || (units - 1) * unit >= words) { std::printf("cut %llu\n", words); return 1; }
    if (snn::raster_scratch(words) < most) { ++over; if (over < 5) std::printf("ring %llu: %llu entries, %llu units\n",
        words, (unsigned long long)snn::raster_scratch(words), most); }
  }
  std::printf("most %llu over %llu\n", most, over);
  return over ? 1 : 0;
}
"""


def test_scratch_holds_the_units_of_every_range(tmp_path):
    src, exe = tmp_path / "units.cpp", tmp_path / "units"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
    assert r.stdout.split()[:2] == ["most", "8192"]
