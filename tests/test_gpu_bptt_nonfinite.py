"""Readout weights and incoming gradients that are not finite, in the event-driven form and in the
general one (more than 2,048 hidden neurons): the readout's sums take every neuron and step,
so 0 times such a value makes them NaN, and what no such value enters is as it is without them."""
import numpy as np
import pytest

from paper_1912_07423_amd import workloads as W
from test_gpu_bptt import _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


def _data(H):
    return W.bptt_inputs(batch=9, steps=70, n_in=30, n_hidden=H, n_out=5, p_in=0.4, p_rec=0.02 if H > 200 else 0.3,
                         rate_lo=60.0, rate_hi=200.0, seed=8)


@pytest.mark.parametrize("H", [40, 130, 2050])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_readout_weight(H, bad):
    d = _data(H)
    plan, loss, _ = _run(d, 10)
    s, _, m, tm = plan.trace()
    assert np.isfinite(loss)
    silent = int(np.argmin(s.sum(axis=(0, 1))))   # spikes in no or few steps
    w = d["w_out"].copy()
    w[silent, 3] = bad
    d["w_out"] = w
    plan2, loss2, _ = _run(d, 10)
    s2, _, m2, tm2 = plan2.trace()
    assert np.array_equal(s, s2)
    assert np.isnan(loss2) and np.isnan(m2[:, 3]).all()
    keep = [0, 1, 2, 4]
    assert np.array_equal(m[:, keep], m2[:, keep]) and np.array_equal(tm[:, keep], tm2[:, keep])


@pytest.mark.parametrize("H", [40, 130, 2050])
def test_label_out_of_range(H):
    d = _data(H)
    d["labels"] = d["labels"].copy()
    d["labels"][4] = 5
    plan, loss, (g_in, g_rec, g_out) = _run(d, 10)
    s = plan.trace()[0]
    assert np.isnan(loss)
    # the adjoint of batch element 4 is NaN up to the step of each maximum, for every neuron
    assert s[0, 4].min() == 0 and np.isnan(g_out).all()


@pytest.mark.parametrize("H", [40, 130, 2050])
@pytest.mark.parametrize("scale", [float("inf"), float("nan")])
def test_incoming_gradient(H, scale):
    d = _data(H)
    plan, loss, (g_in, g_rec, g_out) = _run(d, 10, g_scale=scale)
    assert np.isfinite(loss)
    assert np.isnan(g_out).all()
    plan2, loss2, grads = _run(d, 10, g_scale=2.0)
    assert loss2 == loss and all(np.isfinite(g).all() for g in grads)


def test_a_finite_pass_after_one_that_is_not():
    import torch
    d = _data(130)
    plan, loss, want = _run(d, 10)
    dev = plan.device
    v_in, v_rec = plan.csr_values(d["w_in"], d["w_rec"])
    x, y = torch.tensor(d["x"], device=dev), torch.tensor(d["labels"].astype(np.int32), device=dev)
    bad = d["w_out"].copy()
    bad[3, 1] = np.inf
    for w_out, scale in ((bad, 1.0), (d["w_out"], float("inf")), (d["w_out"], 1.0)):
        ws = [torch.tensor(w, device=dev, requires_grad=True) for w in (v_in, v_rec, w_out)]
        out = plan.loss(x, *ws, y)
        got = torch.autograd.grad(out * scale, ws)
    assert out.item() == loss
    for g, w in zip(got, want):
        assert np.array_equal(g.cpu().numpy(), w)
