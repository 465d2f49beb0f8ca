"""Driven members of a batch at the sizes where a workgroup's words do not divide evenly among its
wavefronts, in every launch shape, against networks of their own."""
import numpy as np
import pytest

from paper_1912_07423_amd import Batch
from paper_1912_07423_amd import workloads as W
from gpu_compare import bits, net as _net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


def _specs(sizes):
    return [W.brunel_fixed_out(n=n, k=min(n - 1, 40), delay_steps=1 + n % 3 if n < 10_000 else 1, rate_hz=40.0, j_mV=0.3, seed=n)
            for n in sizes]


# the largest member decides the neurons per lane: 4,096 and 8,192 per workgroup, and more
@pytest.mark.parametrize("sizes", [(2, 63, 64, 65, 300, 1000, 1025, 4095), (130, 4096), (65, 2049, 4097, 8191), (70, 8193),
                                   (1, 20480)])
@pytest.mark.parametrize("block", [256, 512, 1024])
def test_driven_members(sizes, block):
    specs = _specs([max(2, n) for n in sizes])
    b = Batch(specs, raster_steps=64)
    b.set_tuning(block, 4)
    for steps in (30, 1, 33):
        b.run(steps)
    for k, spec in enumerate(specs):
        g, m = _net(spec, raster_steps=64), b.network(k)
        g.run(64)
        assert np.array_equal(g.raster_bits(0, 64), m.raster_bits(0, 64)), sizes[k]
        sg, sm = g.state(), m.state()
        assert np.array_equal(bits(sg["v"]), bits(sm["v"]))
        assert np.array_equal(sg["ref"], sm["ref"]) and np.array_equal(sg["input"], sm["input"])
        assert g.info()["spikes"] == m.info()["spikes"] and (g.info()["spikes"] > 0 or sizes[k] < 63)
