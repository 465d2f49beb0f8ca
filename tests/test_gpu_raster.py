"""The spike download's kernels (sorted (step, id) pairs) against the raster rows, which the
oracle comparisons of the other files pin: ranges on both sides of the one-workgroup form's
limit, rows of less than one word to many, a ring that wraps inside the range, dense rows,
and more spikes than one block of pinned staging holds."""
import numpy as np
import pytest

from paper_1912_07423_amd import workloads as W
from gpu_compare import net as _net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


def _check(g, t0, t1):
    t, i = np.nonzero(g.raster(t0, t1))
    for _ in range(2):  # the second call's arrays are sized from the first
        steps, ids = g.spikes(t0, t1)
        assert steps.dtype == ids.dtype == np.uint32
        assert np.array_equal(steps, t + t0) and np.array_equal(ids, i)
    return len(ids)


def _always(n, **kw):
    """n neurons without synapses, driven far above threshold and never refractory: every
    neuron spikes at every step."""
    return {"params": W.params(v_bg_mV=1e6, t_ref_ms=0.0, **kw), "pops": [{"size": n, "excitatory": 1}],
            "projs": [], "steps": 1}


# 16,384 words (the one-workgroup form's limit) are 256 rows of 4,096 neurons
@pytest.mark.parametrize("n,ring,run,t0,t1", [
    (63, 64, 80, 16, 80), (64, 64, 100, 40, 99), (65, 7, 20, 13, 20),
    (4000, 300, 300, 0, 256), (4096, 300, 300, 0, 256), (4097, 300, 300, 0, 256),
    (20001, 200, 330, 140, 330), (20001, 200, 330, 131, 183), (1000, 3000, 5000, 2001, 5000),
])
def test_pairs_equal_raster_rows(n, ring, run, t0, t1):
    k = min(100, n - 1)
    g = _net(W.brunel_fixed_out(n=n, k=k, delay_steps=3, rate_hz=60.0, seed=n), raster_steps=ring)
    g.run(run)
    count = _check(g, t0, t1)
    assert count > 0 or n < 64


@pytest.mark.parametrize("n,steps", [(1, 64), (64, 5), (130, 300), (4096, 257)])
def test_dense_rows(n, steps):
    g = _net(_always(n), raster_steps=steps)
    g.run(steps)
    assert _check(g, 0, steps) == n * steps


def test_more_spikes_than_a_staging_block():
    n, steps = 20_000, 230  # 4.6e6 pairs: 36.8 MB, where a block holds 32 MiB
    g = _net(_always(n), raster_steps=steps)
    g.run(steps)
    got_steps, got_ids = g.spikes(0, steps)
    assert np.array_equal(got_steps, np.repeat(np.arange(steps), n))
    assert np.array_equal(got_ids, np.tile(np.arange(n), steps))
