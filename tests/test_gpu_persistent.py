"""snn_run of small static networks without drive (the persistent one-workgroup kernel)
against the launch-per-window pipeline, which an explicit delivery selects and the oracle
comparisons of the other files pin, and against the oracle: every launch shape's size limits,
ragged sizes, delays, both weight layouts, step counts that mix the two paths, more spikes per
step than the kernel's LDS queue holds, caller-set refractory counts, and the FIFO ring that
the run leaves."""
import numpy as np
import pytest

import oracle
from paper_1912_07423_amd import workloads as W
from gpu_compare import bits, compare_net, net as _net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


def _spec(n, degree=20, **kw):
    n_inh = max(1, n // 5)
    kw = {"v_bg_mV": 14.0, "seed": n, **kw}
    return W.ei_er(max(1, n - n_inh), n_inh, min(1.0, degree / n), 1.0, -2.0, **kw)


def _queues(g):
    """Queue counters, and every sub-queue's entries in ascending order (the order of the
    appends is not defined)."""
    s, i = g.state(queues=True), g.info()
    cap = i["queue_stride"] // i["queue_groups"]
    rows = [np.sort(q[k * cap:k * cap + c]).tolist() for q, n in zip(s["queue"], s["queue_len"]) for k, c in enumerate(n)]
    return s["queue_len"], rows


def _same(a, b, t):
    ia, ib = a.info(), b.info()
    assert (ia["t"], ia["events"], ia["spikes"]) == (ib["t"], ib["events"], ib["spikes"]) and ia["t"] == t
    held = min(t, ia["raster_steps"])
    assert np.array_equal(a.raster_bits(t - held, t), b.raster_bits(t - held, t))
    sa, sb = a.state(), b.state()
    assert np.array_equal(bits(sa["v"]), bits(sb["v"]))
    assert np.array_equal(sa["ref"], sb["ref"]) and np.array_equal(sa["input"], sb["input"])
    (la, ra), (lb, rb) = _queues(a), _queues(b)
    assert np.array_equal(la, lb) and ra == rb


@pytest.mark.parametrize("n,delay", [(2, 1), (63, 1), (64, 3), (65, 1), (1024, 1), (1025, 2), (4096, 1), (4097, 1),
                                     (8192, 1), (8193, 2), (20480, 1), (20481, 1), (32001, 1), (40700, 1)])
def test_same_as_the_pipeline(n, delay):
    a = _net(_spec(n, delay_steps=delay), raster_steps=128)
    b = _net(_spec(n, delay_steps=delay), raster_steps=128, delivery="atomic")
    t = 0
    for steps in (2, 1, 3, 40, 1, 83):
        a.run(steps)
        b.run(steps)
        t += steps
        _same(a, b, t)
    a.step()
    b.step()
    a.run(2)
    b.run(2)
    _same(a, b, t + 3)
    assert n < 64 or a.events > 0


@pytest.mark.parametrize("n,delay", [(1000, 1), (4000, 2), (9001, 1)])
def test_same_as_the_oracle(n, delay):
    steps = 200
    spec = _spec(n, delay_steps=delay)
    g = _net(spec, raster_steps=steps)
    o = oracle.OracleNet(spec, raster_cap=steps)
    g.run(120)
    g.run(80)
    o.run(steps)
    compare_net(g, o, steps)


def test_weight_per_synapse():
    spec = _spec(3000, delay_steps=1)
    spec["projs"][1]["w_mV"] = 0.7
    a = _net(spec, raster_steps=64)
    b = _net(spec, raster_steps=64, delivery="atomic")
    assert not a.info()["source_weights"]
    a.run(64)
    b.run(64)
    _same(a, b, 64)


@pytest.mark.parametrize("n", [1000, 5003, 30000])
def test_every_neuron_spikes_at_every_step(n):
    """More spikes than LDS queue entries: the rest goes through the network's queue buffer."""
    kw = dict(v_bg_mV=1e6, t_ref_ms=0.0)
    a = _net(_spec(n, degree=6, **kw), raster_steps=16)
    b = _net(_spec(n, degree=6, **kw), raster_steps=16, delivery="atomic")
    for t in (5, 21):
        a.run(t if t == 5 else 16)
        b.run(t if t == 5 else 16)
        _same(a, b, t)
    assert a.info()["spikes"] == 21 * n


def test_refractory_counts_set_by_the_caller():
    n = 500
    a = _net(_spec(n), raster_steps=64)
    b = _net(_spec(n), raster_steps=64, delivery="atomic")
    ref = np.random.default_rng(1).integers(-5, 40, n)
    ref[:3] = (-2**31, 2**31 - 1, 0)
    v = np.full(n, -49.0, np.float32)
    v[::2] = -60.0
    for g in (a, b):
        g.run(2)
        g.set_state(ref=ref, v=v)
        g.run(20)
    _same(a, b, 22)
    for g in (a, b):
        g.run(30)
    _same(a, b, 52)
