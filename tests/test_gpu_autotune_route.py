"""Autotuning the delivery leaves the way in which snn_run advances a network: a route of its own
stays (before and after an explicit choice by the caller), launches stay launches, and the results
are those of an untuned network."""
import numpy as np
import pytest

from paper_1912_07423_amd import workloads as W
from gpu_compare import bits, net as _net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


def _same(a, b):
    ia, ib = a.info(), b.info()
    for k in ("t", "events", "spikes", "touches"):
        assert ia[k] == ib[k], k
    assert np.array_equal(a.raster_bits(ia["t"] - 60, ia["t"]), b.raster_bits(ib["t"] - 60, ib["t"]))
    plastic = bool(ia["plastic"])
    sa, sb = a.state(weights=plastic), b.state(weights=plastic)
    for k in ("v", "x_pre", "x_post") + (("w_f32",) if plastic else ()):
        assert np.array_equal(bits(sa[k]), bits(sb[k])), k
    assert np.array_equal(sa["ref"], sb["ref"])


@pytest.mark.parametrize("spec,way", [
    (W.ei_er(800, 200, 0.05, 0.5, -2.0, v_bg_mV=14.0, seed=1), "persistent"),
    (W.ei_er(400, 100, 0.05, 0.5, -2.0, v_bg_mV=14.0, seed=2, delay_steps=3), "persistent"),
    (W.stdp_er(n=3000, p=0.03, delay_steps=10, rate_hz=60.0), "windows"),
    (W.stdp_er(n=17000, p=0.005, delay_steps=4, rate_hz=60.0), "windows"),
    (W.brunel_fixed_out(n=3000, k=100, delay_steps=8, rate_hz=40.0), "launches"),
])
def test_autotuned_network_keeps_its_route(spec, way):
    a, b = _net(spec, raster_steps=64), _net(spec, raster_steps=64)
    assert a.route() == b.route() == way
    for g in (a, b):
        g.run(70)
    a.autotune_delivery(reps=1)
    assert a.route() == way
    a.step()  # the tuned launches
    b.step()
    for g in (a, b):
        g.run(59)
    _same(a, b)
    a.set_delivery("atomic")  # the caller's choice
    assert a.route() == "launches"
    a.autotune_delivery(reps=1)
    assert a.route() == "launches"
    for g in (a, b):
        g.run(60)
    _same(a, b)
    a.set_delivery("auto")
    a.autotune_delivery(reps=1)
    assert a.route() == way
    for g in (a, b):
        g.run(60)
    _same(a, b)
