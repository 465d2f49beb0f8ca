"""An eagerly plastic network is built wherever its launch-per-phase form fits the device memory:
the buffers of its windows are optional and the first to give way."""
import ctypes as C

import numpy as np
import pytest

from paper_1912_07423_amd import _lib as L
from paper_1912_07423_amd import workloads as W
from paper_1912_07423_amd.network import _structs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


class _Budget:
    """Device memory from torch's caching allocator, `limit` bytes of it."""

    def __init__(self, limit):
        import torch
        self.limit, self.live, self.peak, self.sizes = limit, {}, 0, []

        def _alloc(nbytes, s, ctx):
            if sum(self.live.values()) + nbytes > self.limit:
                return None
            p = torch.cuda.caching_allocator_alloc(int(nbytes))
            self.live[p] = int(nbytes)
            self.sizes.append(int(nbytes))
            self.peak = max(self.peak, sum(self.live.values()))
            return p

        def _free(p, nbytes, s, ctx):
            assert self.live.pop(p) == nbytes
            torch.cuda.caching_allocator_delete(p)

        self.fns = (L.ALLOC_FN(_alloc), L.FREE_FN(_free))
        self.struct = L.Allocator(self.fns[0], self.fns[1], None)


def _build(spec, limit, delivery="auto"):
    """(status, route, spikes of 60 steps, budget) of a network on `limit` bytes."""
    lib, mem = L.load(), _Budget(limit)
    p, pops, projs, n_projs = _structs(spec, raster_steps=64, delivery=L.DELIVERY[delivery])
    h, way, count = C.c_void_p(), C.c_uint32(), C.c_uint64()
    st = lib.snn_build_network(C.byref(p), pops, len(spec["pops"]), projs, n_projs, C.byref(mem.struct), None,
                               C.byref(h))
    found = None
    if st == L.SNN_OK:
        L.check(lib.snn_get_route(h, C.byref(way)))
        L.check(lib.snn_run(h, 60))
        steps, ids = np.zeros(60 * 3000, np.uint32), np.zeros(60 * 3000, np.uint32)
        L.check(lib.snn_get_raster(h, 0, 60, steps.ctypes.data, ids.ctypes.data, len(ids), C.byref(count)))
        found = steps[:count.value].tolist(), ids[:count.value].tolist()
    lib.snn_destroy(h)
    assert not mem.live
    return st, L.ROUTE_NAME[way.value], found, mem


def test_windows_give_way():
    spec = W.stdp_er(n=3000, p=0.05, delay_steps=8, rate_hz=60.0)
    st, way, want, plain = _build(spec, 1 << 40, delivery="atomic")
    assert (st, way) == (L.SNN_OK, "launches") and len(want[0]) > 0
    st, way, found, full = _build(spec, 1 << 40)
    assert (st, way) == (L.SNN_OK, "windows") and found == want
    extra = full.peak - plain.peak
    assert extra > 0
    # from just what the launches need to one byte less than everything
    for part in (0.0, 0.2, 0.4, 0.6, 0.8, 0.95):
        st, way, found, mem = _build(spec, plain.peak + int(part * extra))
        assert (st, way) == (L.SNN_OK, "launches"), (part, way)
        assert found == want
    st, way, found, mem = _build(spec, full.peak - 1)
    assert (st, way) == (L.SNN_OK, "launches") and found == want
    st, way, found, mem = _build(spec, full.peak)
    assert (st, way) == (L.SNN_OK, "windows") and found == want
    assert _build(spec, plain.peak - 1)[0] == L.SNN_E_OOM
