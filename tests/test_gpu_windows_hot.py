"""Windows of eagerly plastic networks whose lane groups are chosen for many spikes (more than about
50,000 neurons): sub-rows longer than a lane group, more of them in a step than are in flight, more in
a window than are laid out, against the launch-per-phase pipeline."""
import numpy as np
import pytest

from paper_1912_07423_amd import workloads as W
from gpu_compare import bits, net as _net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


# mean synapses per sub-row: 1.5 in 4 lanes, 5.1 in 8, 8.9 in 16
@pytest.mark.parametrize("n,degree,delay", [(140_000, 420, 10), (60_000, 1200, 17), (100_000, 2000, 4)])
def test_many_spikes(n, degree, delay):
    print(f"[windows] hot n={n} degree={degree} d={delay}", flush=True)
    spec = W.stdp_er(n=n, p=degree / n, delay_steps=delay, rate_hz=100.0, seed=n)
    a, b = _net(spec, raster_steps=64), _net(spec, raster_steps=64, delivery="tiled")
    assert (a.route(), b.route()) == ("windows", "launches")
    for steps in (40, 7, 64):
        for g in (a, b):
            g.run(steps)
        ia, ib = a.info(), b.info()
        for k in ("t", "events", "spikes", "touches"):
            assert ia[k] == ib[k], k
        t = ia["t"]
        held = min(t, 64)
        assert np.array_equal(a.raster_bits(t - held, t), b.raster_bits(t - held, t))
    assert ia["spikes"] / t > n * 0.003  # over 30 Hz
    sa, sb = a.state(weights=True), b.state(weights=True)
    for k in ("v", "x_pre", "x_post", "w_f32"):
        assert np.array_equal(bits(sa[k]), bits(sb[k])), k
    assert np.array_equal(sa["ref"], sb["ref"]) and np.array_equal(sa["input"], sb["input"])
