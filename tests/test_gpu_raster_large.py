"""Spike download from rings of more than 4,194,304 words, with ranges that are cut into more
units than the whole ring: the pairs equal the raster rows, and a network that was made next to
the ring keeps its state."""
import numpy as np
import pytest

from paper_1912_07423_amd import workloads as W
from gpu_compare import bits, net as _net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


@pytest.mark.parametrize("n,ring,rows", [(300_000, 1024, 1000), (262_208, 1024, 1023)])
def test_range_with_more_units_than_its_ring(n, ring, rows):
    g = _net(W.brunel_fixed_out(n=n, k=4, delay_steps=15, rate_hz=20.0, seed=3), raster_steps=ring)
    other = _net(W.brunel_fixed_out(n=5000, k=100, delay_steps=15, seed=4), raster_steps=64)
    g.run(ring)
    other.run(64)
    before = other.state(queues=True)
    steps, ids = g.spikes(ring - rows, ring)
    words = g.raster_bits(ring - rows, ring)
    t, w = np.nonzero(words)  # few words hold a spike
    want = np.unpackbits(words[t, w].view(np.uint8).reshape(-1, 8), axis=1, bitorder="little")
    k, b = np.nonzero(want)
    assert len(ids) > 0
    assert np.array_equal(steps, t[k] + (ring - rows)) and np.array_equal(ids, w[k] * 64 + b)
    after = other.state(queues=True)
    for key in before:
        x, y = np.asarray(before[key]), np.asarray(after[key])
        assert np.array_equal(bits(x), bits(y)) if x.dtype == np.float32 else np.array_equal(x, y), key
    g.run(2)  # the control block and drive tables behind the ring
    assert g.info()["t"] == ring + 2
