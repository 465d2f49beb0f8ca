"""The busy form of the event-driven plans' forward pass (a launch per step, for passes with many
spikes) against the quiet one, which the oracle comparisons of the other files pin: the same
trajectory, loss and gradients bit for bit, at one to five wavefronts of neurons' rows, batches below and at a
wavefront, step counts around the sampling, rows that fit the padded copy or do not, inputs
other than 0 and 1, and with the steps launched one by one.  And the choice between the two: by
the activity of finished passes, in both directions."""
import math

import numpy as np
import pytest

from paper_1912_07423_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu_available):
    return gpu_available


class _Plan:
    def __init__(self, d, theta, **kw):
        import torch
        from paper_1912_07423_amd.bptt import RecurrentLIF
        B, T, _ = d["x"].shape
        H, O = d["w_out"].shape
        self.torch, self.plan = torch, RecurrentLIF(d["mask_in"], d["mask_rec"], O, B, T, checkpoint=7, theta=theta, **kw)
        self.w = [torch.tensor(w, device="cuda", requires_grad=True)
                  for w in (*self.plan.csr_values(d["w_in"], d["w_rec"]), d["w_out"])]
        self.y = torch.tensor(d["labels"].astype(np.int32), device="cuda")

    def run(self, x):
        """(route, loss, gradients, trace) of one iteration, finished."""
        torch = self.torch
        way = self.plan.route()
        loss = self.plan.loss(torch.tensor(x, device="cuda"), *self.w, self.y)
        g = torch.autograd.grad(loss, self.w)
        torch.cuda.synchronize()
        return way, loss.item(), [t.cpu().numpy() for t in g], self.plan.trace()


def _same(a, b):
    assert a[1] == b[1]
    for x, y in zip(a[2], b[2]):
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32))
    for x, y in zip(a[3], b[3]):
        assert np.array_equal(x, y)


def _data(B, T, C, H, O, p_in=0.4, p_rec=0.1, seed=51):
    d = W.bptt_inputs(batch=B, steps=T, n_in=C, n_hidden=H, n_out=O, p_in=p_in, p_rec=p_rec, rate_lo=200.0,
                      rate_hi=600.0, seed=seed)
    d["w_in"] = np.abs(d["w_in"]) * 2
    return d


@pytest.mark.parametrize("B,T,C,H,p_rec", [
    (64, 60, 40, 400, 0.1), (9, 33, 65, 256, 0.3), (1, 40, 30, 257, 0.3), (64, 17, 12, 1024, 0.05), (33, 20, 20, 1025, 0.05),
    (5, 16, 12, 2048, 0.02), (64, 30, 40, 300, 0.95), (7, 5, 25, 200, 0.5), (8, 3, 25, 200, 0.5), (64, 2, 25, 200, 0.5)])
@pytest.mark.parametrize("eager", [False, True])
def test_busy_equals_quiet(B, T, C, H, p_rec, eager):
    d = _data(B, T, C, H, 3, p_rec=p_rec)
    p = _Plan(d, theta=0.02, eager=eager)
    first = p.run(d["x"])
    assert first[0] == "persistent"
    second = p.run(d["x"])
    assert second[0] == "launches"
    third = p.run(d["x"])  # replayed
    assert third[0] == "launches"
    _same(first, second)
    _same(first, third)
    assert first[3][0].sum() > 0.2 * B * T * H


def test_real_valued_inputs():
    d = _data(20, 40, 30, 300, 4)
    d["x"] = (d["x"] * np.random.default_rng(1).random(d["x"].shape)).astype(np.float32)
    p = _Plan(d, theta=0.02)
    first, second = p.run(d["x"]), p.run(d["x"])
    assert (first[0], second[0]) == ("persistent", "launches")
    _same(first, second)


def test_the_route_follows_the_activity():
    d = _data(32, 50, 60, 500, 4)
    quiet = np.zeros_like(d["x"])
    quiet[:, -3:, 0] = 1  # the recurrent input keeps itself up otherwise
    p, ref = _Plan(d, theta=0.02), _Plan(d, theta=0.02)
    want_busy = ref.run(d["x"])
    want_quiet = _Plan(d, theta=0.02).run(quiet)
    assert p.plan.route() == "persistent"
    for x, want, after in ((quiet, want_quiet, "persistent"), (d["x"], want_busy, "launches"), (d["x"], want_busy, "launches"),
                           (quiet, want_quiet, "persistent"), (quiet, want_quiet, "persistent"),
                           (d["x"], want_busy, "launches")):
        _same(p.run(x), want)
        assert p.plan.route() == after


def test_general_plans_take_the_launches():
    import torch  # noqa: F401
    d = _data(4, 6, 10, 40, 2)
    assert _Plan(d, theta=1.0, smooth=True).plan.route() == "launches"


def test_captured_busy_pass():
    """A plan whose latest pass was busy, captured into the caller's graph: the quiet form, as the
    plan's own graph cannot be launched there; replays equal the eager result."""
    import torch
    d = _data(16, 20, 30, 300, 3)
    p = _Plan(d, theta=0.02)
    x = torch.tensor(d["x"], device="cuda")
    s = torch.cuda.Stream()
    ws = [w.detach() for w in p.w]
    with torch.cuda.stream(s), torch.no_grad():
        for _ in range(2):
            p.plan.loss(x, *ws, p.y)
            s.synchronize()
        assert p.plan.route() == "launches"
        want = p.plan.loss(x, *ws, p.y).item()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            out = p.plan.loss(x, *ws, p.y)
        for _ in range(3):
            g.replay()
            s.synchronize()
            assert out.item() == want
            assert p.plan.loss(x, *ws, p.y).item() == want
            s.synchronize()


def test_plans_made_and_closed_with_the_caches_released():
    """Every plan reads its own passes' activity: a new plan starts quiet although a busy one has
    just been closed, and more plans at once than one block of slots serves keep theirs apart."""
    from paper_1912_07423_amd.network import memory_cache_release
    d = _data(8, 20, 20, 400, 2)
    want = None
    for release in (False, True, False):
        p = _Plan(d, theta=0.02)
        first = p.run(d["x"])
        assert first[0] == "persistent" and p.plan.route() == "launches"
        want = want or first
        _same(first, want)
        p.plan.close()
        if release:
            memory_cache_release()
    small = _data(2, 4, 6, 20, 2)
    plans = [_Plan(d, theta=0.02)] + [_Plan(small, theta=10.0) for _ in range(70)]
    plans[0].run(d["x"])
    memory_cache_release()
    assert plans[0].plan.route() == "launches" and all(q.plan.route() == "persistent" for q in plans[1:])
    _same(plans[0].run(d["x"]), want)
    for q in plans:
        q.plan.close()
    memory_cache_release()
    _same(_Plan(d, theta=0.02).run(d["x"]), want)
