"""Which way snn_run advances a network (Network.route): the networks whose comparison with the
launch-per-window pipeline means something only if they do not take it themselves, and the
settings that send a network to the launches.  And eagerly plastic windows of more ranges than a
workgroup of the row layout holds boundaries for."""
import numpy as np
import pytest

from paper_1912_07423_amd import _lib as L
from paper_1912_07423_amd import Batch
from paper_1912_07423_amd import workloads as W
from gpu_compare import bits, net as _net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


def _static(n, degree=20, **kw):
    n_inh = max(1, n // 5)
    return W.ei_er(max(1, n - n_inh), n_inh, min(1.0, degree / n), 1.0, -2.0, **{"v_bg_mV": 14.0, "seed": n, **kw})


def _plastic(n, degree, delay, **kw):
    return W.stdp_er(n=n, p=min(1.0, degree / n), delay_steps=delay, **{"rate_hz": 60.0, "seed": n + delay, **kw})


@pytest.mark.parametrize("n,delay", [(2, 1), (63, 1), (1024, 1), (1025, 2), (4096, 1), (4097, 1), (8193, 2)])
def test_small_static_networks_are_persistent(n, delay):
    assert _net(_static(n, delay_steps=delay), raster_steps=16).route() == "persistent"
    assert _net(_static(n, delay_steps=delay), raster_steps=16, delivery="atomic").route() == "launches"


@pytest.mark.parametrize("n,degree,delay", [(2, 2, 5), (3, 3, 2), (63, 20, 3), (1000, 60, 64), (4097, 90, 10),
                                            (16385, 140, 2), (33000, 150, 15)])
def test_eagerly_plastic_networks_run_in_windows(n, degree, delay):
    assert _net(_plastic(n, degree, delay), raster_steps=16).route() == "windows"
    assert _net(_plastic(n, degree, delay), raster_steps=16, delivery="tiled").route() == "launches"


def test_what_takes_the_launches():
    assert _net(_plastic(1000, 60, 1), raster_steps=16).route() == "launches"               # no window
    assert _net(_plastic(1000, 60, 8), raster_steps=16, plasticity="lazy").route() == "launches"
    assert _net(W.brunel_fixed_out(n=1000, k=50), raster_steps=16).route() == "launches"    # driven
    for spec, way in ((_static(1000), "persistent"), (_plastic(1000, 60, 8), "windows")):
        g = _net(spec, raster_steps=16)
        g.set_profiling(True)
        assert g.route() == "launches"
        g.set_profiling(False)
        assert g.route() == way
        g.set_delivery("atomic")
        assert g.route() == "launches"
        g.set_delivery("auto")
        assert g.route() == way


def test_a_batch_member_has_none():
    b = Batch([_static(100), _static(200)], raster_steps=16)
    with pytest.raises(L.SnnError):
        b.network(1).route()


def test_windows_of_more_than_512_ranges():
    """263,000 neurons in 514 ranges of 512: the row layout reads range boundaries from memory."""
    spec = _plastic(263_000, 300, 6, rate_hz=30.0)
    print("[routes] 263k plastic", flush=True)
    a, b = _net(spec, raster_steps=64), _net(spec, raster_steps=64, delivery="atomic")
    assert (a.route(), b.route()) == ("windows", "launches")
    for steps in (40, 3, 41):
        a.run(steps)
        b.run(steps)
        ia, ib = a.info(), b.info()
        for k in ("t", "events", "spikes", "touches"):
            assert ia[k] == ib[k], k
        assert np.array_equal(a.raster_bits(ia["t"] - steps, ia["t"]), b.raster_bits(ib["t"] - steps, ib["t"]))
    sa, sb = a.state(weights=True), b.state(weights=True)
    for k in ("v", "x_pre", "x_post", "w_f32"):
        assert np.array_equal(bits(sa[k]), bits(sb[k])), k
    assert np.array_equal(sa["ref"], sb["ref"]) and np.array_equal(sa["input"], sb["input"])
    assert ia["touches"] > 0
