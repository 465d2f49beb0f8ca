"""The route of a small static network follows its rate where the rate decides which way is the
faster.  Until a call that waits for the device has counted spikes, the first 512 steps take the
persistent kernel and later ones the way that risks less; then the persistent kernel serves at a
low rate, the launches at a high one, and back.  The results do not depend on it."""
import numpy as np
import pytest

from paper_1912_07423_amd import workloads as W
from gpu_compare import bits, net as _net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


def _spec(n, degree, v_bg, w_inh=-0.1, **kw):
    n_inh = n // 5
    return W.ei_er(n - n_inh, n_inh, degree / n, 0.05, w_inh, v_bg_mV=v_bg, seed=n, **kw)


def _quiet(n, degree):
    """Inhibition takes 40 times what excitation gives: a few Hz."""
    return _spec(n, degree, 11.0, w_inh=-8.0)


def _same(a, b):
    ia, ib = a.info(), b.info()
    for k in ("t", "events", "spikes"):
        assert ia[k] == ib[k], k
    held = min(ia["t"], ia["raster_steps"])
    assert np.array_equal(a.raster_bits(ia["t"] - held, ia["t"]), b.raster_bits(ib["t"] - held, ib["t"]))
    sa, sb = a.state(), b.state()
    assert np.array_equal(bits(sa["v"]), bits(sb["v"]))
    assert np.array_equal(sa["ref"], sb["ref"]) and np.array_equal(sa["input"], sb["input"])


def _know(g, how):
    """A call that waits for the device, of each kind."""
    t = g._t
    if how == "sync":
        g.sync()
    elif how == "info":
        assert g.info()["t"] == t
    else:
        g.spikes(t - 64, t)


def _advance(nets, steps):
    for g in nets:
        g.run(steps)
        g._t = getattr(g, "_t", 0) + steps


@pytest.mark.parametrize("how", ["sync", "info", "spikes"])
@pytest.mark.parametrize("n,degree", [(16000, 320), (24000, 200), (32001, 300), (40700, 60)])
def test_route_follows_the_rate(n, degree, how):
    print(f"[route] n={n} degree={degree} {how}", flush=True)
    a, b = _net(_spec(n, degree, 60.0), raster_steps=128), _net(_spec(n, degree, 60.0), raster_steps=128, delivery="atomic")
    assert a.route() == "persistent"  # nothing counted yet
    _advance((a, b), 100)
    assert a.route() == "persistent"
    _know(a, how)
    assert a.route() == "launches"  # some 100 Hz
    # refractory for 200 steps: no spikes
    for g in (a, b):
        g.set_state(ref=np.full(n, 200, np.int32))
    _advance((a, b), 130)
    _know(a, how)
    assert a.route() == "persistent"
    _advance((a, b), 10)
    _same(a, b)
    assert a.route() == "persistent"
    _advance((a, b), 130)  # across the end of the silence
    _know(a, how)
    assert a.route() == "launches"
    _advance((a, b), 3)
    _same(a, b)


@pytest.mark.parametrize("n,degree", [(16000, 320), (20480, 100), (20481, 100), (32001, 300), (40700, 60)])
def test_large_persistent_networks_equal_the_pipeline(n, degree):
    """At a low rate, on the persistent kernel's larger launch shapes."""
    a, b = _net(_quiet(n, degree), raster_steps=128), _net(_quiet(n, degree), raster_steps=128, delivery="atomic")
    _advance((a, b), 100)
    a.sync()
    for steps in (2, 70, 3, 200):
        assert a.route() == "persistent"
        _advance((a, b), steps)
        _same(a, b)
    assert a.info()["spikes"] > 0


def test_downloads_of_few_steps_add_up():
    a = _net(_spec(32001, 300, 60.0), raster_steps=64)
    for k in range(7):
        assert a.route() == "persistent"
        a.run(10)
        a.spikes(10 * k, 10 * k + 10)
    assert a.route() == "launches"


@pytest.mark.parametrize("n,degree,then", [(24000, 200, "persistent"), (32001, 300, "launches")])
@pytest.mark.parametrize("steps", [(512,), (511, 2), (513,), (700,)])
def test_first_steps(n, degree, then, steps):
    """Around the 512th step and across it, nothing counted."""
    a, b = _net(_spec(n, degree, 60.0), raster_steps=128), _net(_spec(n, degree, 60.0), raster_steps=128, delivery="atomic")
    for k in steps:
        assert a.route() == "persistent"
        _advance((a, b), k)
    assert a.route() == then
    _same(a, b)


def test_a_network_that_is_faster_at_any_rate_does_not_count():
    a = _net(W.cuba_lif_4k(v_bg_mV=60.0), raster_steps=64)
    assert a.route() == "persistent"
    a.run(100)
    a.sync()
    assert a.route() == "persistent"


def test_a_rate_that_changes_late_is_noticed():
    """After many counts that confirmed the route, within 4,096 steps."""
    n = 32001
    a = _net(_quiet(n, 300), raster_steps=128)
    for _ in range(60):
        a.run(100)
        a.sync()
    assert a.route() == "persistent"
    for _ in range(48):
        a.set_state(v=np.full(n, 100.0, np.float32), ref=np.zeros(n, np.int32))  # all spike
        a.run(100)
        a.sync()
    assert a.route() == "launches"
