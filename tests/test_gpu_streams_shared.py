"""Batches and training plans take the kept streams of closed objects, as networks do: objects of
all three kinds made, run and closed by several threads at once give the results they give alone."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from paper_1912_07423_amd import Batch
from paper_1912_07423_amd import workloads as W
from gpu_compare import net as _net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


def _network(seed):
    with _net(W.brunel_fixed_out(n=1200, k=50, delay_steps=4, rate_hz=30.0, j_mV=0.5, seed=seed), raster_steps=128,
              torch_memory=False) as g:
        g.run(100)
        return g.spikes(0, 100)


def _batch(seed):
    specs = [W.ei_er(400, 100, 0.05, 0.5, -2.0, v_bg_mV=14.0, seed=seed + k) for k in range(3)]
    with Batch(specs, raster_steps=128, torch_memory=False) as b:
        b.run(100)
        return b.network(1).spikes(0, 100)


def _plan(seed):
    import torch
    from paper_1912_07423_amd.bptt import RecurrentLIF
    d = W.bptt_inputs(batch=5, steps=30, n_in=20, n_hidden=70, n_out=3, p_in=0.4, p_rec=0.2, rate_lo=80.0, rate_hi=200.0,
                      seed=seed)
    p = RecurrentLIF(d["mask_in"], d["mask_rec"], 3, 5, 30)
    w = [torch.tensor(x, device="cuda", requires_grad=True) for x in (*p.csr_values(d["w_in"], d["w_rec"]), d["w_out"])]
    x, y = torch.tensor(d["x"], device="cuda"), torch.tensor(d["labels"].astype(np.int32), device="cuda")
    torch.cuda.synchronize()  # the plan's own stream is not torch's
    loss = p.loss(x, *w, y)
    torch.cuda.synchronize()
    g = torch.autograd.grad(loss, w)
    torch.cuda.synchronize()
    out = [loss.detach().cpu().numpy(), *(t.cpu().numpy() for t in g)]
    p.close()
    return out


def _same(a, b):
    return len(a) == len(b) and all(np.array_equal(x, y) for x, y in zip(a, b))


def test_objects_of_all_kinds_share_the_kept_streams():
    jobs = [(f, s) for s in range(1, 5) for f in (_network, _batch, _plan)]
    alone = [f(s) for f, s in jobs]
    for _ in range(2):  # one after another on the streams kept by then
        assert all(_same(f(s), w) for (f, s), w in zip(jobs, alone))
    with ThreadPoolExecutor(6) as pool:
        for _ in range(2):
            got = list(pool.map(lambda j: j[0](j[1]), [j for j in jobs if j[0] is not _plan] * 2))
            assert all(_same(g, w) for g, w in zip(got, [w for j, w in zip(jobs, alone) if j[0] is not _plan] * 2))
