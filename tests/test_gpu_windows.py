"""snn_run of eagerly plastic networks with a delay of at least two steps (windows of steps in
one launch) against the launch-per-phase pipeline, which an explicit delivery selects, and
against the oracle: ragged sizes around a wavefront and around the ranges of targets, delays
around the longest window, step counts that mix both paths, more arriving spikes than a
workgroup's LDS list holds, queues written by the caller, and a delivery chosen later.  All
results must be the same bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1912_07423_amd import workloads as W
from gpu_compare import bits, compare_net, net as _net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


def _spec(n, degree, delay, **kw):
    kw = {"rate_hz": 60.0, "n_ext": 1000, "seed": n + delay, **kw}
    return W.stdp_er(n=n, p=min(1.0, degree / n), delay_steps=delay, **kw)


def _queues(g):
    """The queues still to arrive: S of the last `delay` steps, ascending in every sub-queue
    (the order of the appends is not defined), and the empty queue of the next step."""
    s, i = g.state(queues=True), g.info()
    cap, t = i["queue_stride"] // i["queue_groups"], i["t"]
    rows = []
    for step in list(range(max(0, t - i["delay"]), t)) + [t]:
        q, n = s["queue"][step % i["queue_slots"]], s["queue_len"][step % i["queue_slots"]]
        rows.append([np.sort(q[k * cap:k * cap + c]).tolist() for k, c in enumerate(n)])
    assert rows[-1] == [[]] * i["queue_groups"]
    return rows


def _same(a, b):
    ia, ib = a.info(), b.info()
    for k in ("t", "events", "spikes", "touches"):
        assert ia[k] == ib[k], k
    t = ia["t"]
    held = min(t, ia["raster_steps"])
    assert np.array_equal(a.raster_bits(t - held, t), b.raster_bits(t - held, t))
    sa, sb = a.state(weights=True), b.state(weights=True)
    for k in ("v", "x_pre", "x_post", "w_f32"):
        assert np.array_equal(bits(sa[k]), bits(sb[k])), k
    assert np.array_equal(sa["ref"], sb["ref"]) and np.array_equal(sa["input"], sb["input"])
    assert _queues(a) == _queues(b)


@pytest.mark.parametrize("n,degree,delay", [(2, 2, 5), (3, 3, 2), (63, 20, 3), (64, 20, 2), (65, 20, 4), (1000, 60, 17),
                                            (1000, 60, 18), (1000, 60, 64), (4097, 90, 10), (16384, 140, 7),
                                            (16385, 140, 2), (33000, 150, 15)])
def test_same_as_the_pipeline(n, degree, delay):
    print(f"[windows] n={n} d={delay}", flush=True)
    a = _net(_spec(n, degree, delay), raster_steps=128)
    b = _net(_spec(n, degree, delay), raster_steps=128, delivery="atomic")
    for steps in (2, 1, 3, 40, 1, 1, 83):
        a.run(steps)
        b.run(steps)
        _same(a, b)
    a.step()
    b.step()
    a.run(delay)
    b.run(delay)
    _same(a, b)
    assert n < 63 or (a.info()["events"] > 0 and a.info()["touches"] > 0)


@pytest.mark.parametrize("n,degree,delay,kw", [
    (777, 62, 2, {}), (2000, 100, 10, {}), (600, 60, 3, {"rate_hz": 400.0, "n_ext": 200}),
    (9001, 100, 6, {"rate_hz": 0.0, "n_ext": 0})])
def test_same_as_the_oracle(n, degree, delay, kw):
    steps = 300
    spec = _spec(n, degree, delay, **kw)
    print(f"[windows] oracle n={n} d={delay}", flush=True)
    g = _net(spec, raster_steps=steps)
    o = oracle.OracleNet(spec, raster_cap=steps)
    g.run(170)
    g.run(130)
    o.run(steps)
    compare_net(g, o, steps)


def test_smallest_raster_ring():
    spec = _spec(1500, 75, 9)
    a, b = _net(spec, raster_steps=1), _net(spec, raster_steps=1, delivery="tiled")
    assert a.info()["raster_steps"] == 10
    for steps in (5, 50, 9):
        a.run(steps)
        b.run(steps)
        _same(a, b)


def test_neurons_that_fire_in_consecutive_steps():
    """No refractory time and a strong drive: most neurons fire at most steps, so rows are
    depressed and delivered in the same step, and a window's arrivals exceed a workgroup's
    LDS list many times over."""
    spec = _spec(3000, 90, 6, rate_hz=400.0, n_ext=200)
    spec["params"].update(t_ref_ms=0.0, w_ext_mV=2.0)
    a, b = _net(spec, raster_steps=64), _net(spec, raster_steps=64, delivery="atomic")
    for steps in (30, 2, 30):
        a.run(steps)
        b.run(steps)
        _same(a, b)
    i = a.info()
    assert i["spikes"] > 62 * 1000  # of 3,000 neurons; a list holds 2,048 spikes of a window


def test_queues_written_by_the_caller():
    """A state whose pending queues differ from the recorded spikes is stepped as the
    launches step it until the queues have arrived."""
    spec = _spec(1200, 70, 8)
    a, b = _net(spec, raster_steps=64), _net(spec, raster_steps=64, delivery="atomic")
    a.run(40)
    b.run(40)
    s = b.state(queues=True)
    cap = b.info()["queue_stride"] // b.info()["queue_groups"]
    slot = 37 % b.info()["queue_slots"]
    s["queue"][slot, :cap][:3] = (5, 6, 7)
    s["queue_len"][slot, 0] = 3
    for g in (a, b):
        g.set_state(queue=s["queue"], queue_len=s["queue_len"])
    for steps in (3, 4, 30):
        a.run(steps)
        b.run(steps)
        _same(a, b)


def test_delivery_chosen_later():
    spec = _spec(2500, 80, 5)
    a, b = _net(spec, raster_steps=64), _net(spec, raster_steps=64, delivery="atomic")
    for kind in ("auto", "tiled", "auto", "atomic", "auto"):
        a.set_delivery(kind)
        a.run(33)
        b.run(33)
        _same(a, b)
    c, d = _net(spec, raster_steps=64, delivery="tiled"), _net(spec, raster_steps=64, delivery="atomic")
    c.run(20)
    c.set_delivery("auto")
    c.run(45)
    d.run(65)
    _same(c, d)


def test_profiled_steps_between():
    spec = _spec(2500, 80, 5)
    a, b = _net(spec, raster_steps=64), _net(spec, raster_steps=64, delivery="atomic")
    for on in (True, False, True, False):
        a.set_profiling(on)
        a.run(33)
        b.run(33)
        a.set_profiling(False)
        _same(a, b)
