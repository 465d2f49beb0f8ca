"""Update windows of five and more steps of static networks (the inputs of the steps prepared by
several wavefronts, the membranes stepped by one) against one-step windows, which take the plain
form, and against the oracle: sizes around a wavefront and around the largest network of the
split form, windows around its LDS buffer of 20 steps, with and without drive, both deliveries
and every position of the first step in its quad.  Everything must be the same bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1912_07423_amd import workloads as W
from gpu_compare import bits, compare_net, net as _net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


def _spec(n, delay, drive):
    # the excitatory half drives; inhibition keeps the rate of the larger networks moderate
    s = W.brunel_fixed_out(n=n, k=min(40, n - 1), delay_steps=delay, rate_hz=20.0 if drive else 0.0,
                           n_ext=1000 if drive else 0, j_mV=0.4, seed=n + delay)
    if not drive:
        s["params"]["v_bg_mV"] = 14.0
    return s


def _same(a, b):
    ia, ib = a.info(), b.info()
    assert (ia["t"], ia["spikes"]) == (ib["t"], ib["spikes"])
    t = ia["t"]
    assert np.array_equal(a.raster_bits(0, t), b.raster_bits(0, t))
    sa, sb = a.state(), b.state()
    assert np.array_equal(bits(sa["v"]), bits(sb["v"])) and np.array_equal(sa["ref"], sb["ref"])


@pytest.mark.parametrize("drive", [True, False])
@pytest.mark.parametrize("n,delay", [(2, 5), (63, 20), (64, 17), (65, 18), (1000, 64), (4097, 21), (16385, 40),
                                     (81920, 15), (81921, 15)])
def test_same_as_single_steps(n, delay, drive):
    print(f"[update window] n={n} d={delay} drive={drive}", flush=True)
    kw = dict(raster_steps=512, delivery="atomic")
    a, b = _net(_spec(n, delay, drive), **kw), _net(_spec(n, delay, drive), window=1, **kw)
    for steps in (delay, 6, 5, 7, 3 * delay + 1, 130):
        a.run(steps)
        b.run(steps)
    _same(a, b)
    assert n < 63 or a.info()["spikes"] > 0


@pytest.mark.parametrize("delivery", ["atomic", "tiled"])
@pytest.mark.parametrize("n,delay", [(1500, 9), (3001, 23)])
def test_same_as_the_oracle(n, delay, delivery):
    steps = 200
    spec = _spec(n, delay, True)
    g = _net(spec, raster_steps=steps, delivery=delivery)
    o = oracle.OracleNet(spec, raster_cap=steps)
    g.run(steps)
    o.run(steps)
    compare_net(g, o, steps)
