"""Streams of closed networks serve later ones: networks built, run and closed by several threads
at once, more of them open than streams are kept, with the kept streams released in between."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from paper_1912_07423_amd import _lib as L
from paper_1912_07423_amd import workloads as W
from gpu_compare import net as _net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


def _run(seed):
    spec = W.brunel_fixed_out(n=1500, k=60, delay_steps=6, rate_hz=30.0, j_mV=0.5, seed=seed)
    with _net(spec, raster_steps=256, torch_memory=False) as g:
        g.run(70)    # a short first run, launched directly
        g.run(130)   # from a captured graph
        return g.spikes(0, 200)


def test_networks_of_several_threads_share_the_kept_streams():
    seeds = list(range(1, 13)) * 2
    alone = {s: _run(s) for s in set(seeds)}
    with ThreadPoolExecutor(12) as pool:
        for _ in range(2):
            for s, (steps, ids) in zip(seeds, pool.map(_run, seeds)):
                assert len(ids) and np.array_equal(steps, alone[s][0]) and np.array_equal(ids, alone[s][1])
            L.check(L.load().snn_memory_cache_release(-1))
