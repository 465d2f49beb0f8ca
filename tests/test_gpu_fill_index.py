"""Delivery indexes written during the synapse fill (networks whose populations have one
fixed out-degree projection each) against the index pass, which set_delivery runs, and against
the atomic delivery, which needs none: out-degrees around the block of four targets, around the
shortest rows that are filled by workgroups and at their limit, rows without synapses, targets
past 65,536, one tile and many, both weight layouts.  All runs must be the same bit for bit."""
import numpy as np
import pytest

from paper_1912_07423_amd import workloads as W
from gpu_compare import bits, net as _net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


def _spec(n, k, empty=False):
    s = W.brunel_fixed_out(n=n, k=k, delay_steps=7, rate_hz=40.0, j_mV=8.0 / max(8, k), seed=n + k)
    s["params"]["w_ext_mV"] = 0.2
    if empty:  # the inhibitory population projects nowhere
        s["projs"] = s["projs"][:1]
    return s


def _same(nets, steps):
    for g in nets:
        g.run(steps)
    a = nets[0]
    ia, sa = a.info(), a.state()
    ra = a.raster_bits(0, ia["t"])
    for b in nets[1:]:
        ib, sb = b.info(), b.state()
        assert (ia["events"], ia["spikes"]) == (ib["events"], ib["spikes"]) and ia["spikes"] > 0
        assert np.array_equal(ra, b.raster_bits(0, ib["t"]))
        assert np.array_equal(bits(sa["v"]), bits(sb["v"])) and np.array_equal(sa["input"], sb["input"])


_SIZES = [(40, 1, 1), (1000, 2, 3), (1000, 3, 60), (1003, 4, 7), (2000, 5, 125), (3000, 255, 1), (3000, 256, 31),
          (3001, 257, 187), (5000, 1003, 87), (5000, 4095, 20), (6000, 4096, 1), (6000, 4097, 100),
          (6000, 5999, 375), (70001, 130, 0), (140000, 66, 0)]


@pytest.mark.parametrize("n,k,tiles,weights", [(*s, "auto") for s in _SIZES] + [(*s, "per_synapse") for s in _SIZES[-7:]])
def test_same_runs(n, k, tiles, weights):
    print(f"[fill index] n={n} k={k} tiles={tiles} {weights}", flush=True)
    kw = dict(raster_steps=128, synapse_weights=weights)
    a = _net(_spec(n, k), delivery="atomic", **kw)
    b = _net(_spec(n, k), delivery="tiled", tiles=tiles, **kw)
    c = _net(_spec(n, k), delivery="atomic", **kw)
    c.set_delivery("tiled", tiles=tiles)
    _same([a, b, c], 90)


def test_rows_without_synapses():
    kw = dict(raster_steps=128)
    spec = _spec(4000, 200, empty=True)
    _same([_net(spec, delivery="atomic", **kw), _net(spec, delivery="tiled", **kw)], 90)
