"""Calls captured into the caller's own graph, with eager calls on the same
operator before and after its replays: what a replay writes into the
operator's plan is not taken for what the next eager call needs."""
import numpy as np
import pytest

from gpu_common import to_dev
from paper_2108_04315_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,s", [(20, 30, 2), (25, 17, 3)])
def test_eager_calls_around_a_captured_one(h, w, s):
    import torch
    from paper_2108_04315_amd import misr
    ctx = misr.Context(0)
    rng = np.random.default_rng(h)
    shifts = np.array([(0.0, 0.0), (0.45, -0.3)])
    op = misr.Operator(ctx, s * h, s * w, s, shifts, synth.psf_taps(0.8, 7))
    prm = misr.default_params()
    xa, xb = (to_dev(rng.uniform(0, 1, (s * h, s * w))) for _ in range(2))
    ya, yb = (to_dev(rng.uniform(0, 1, (2, h, w))) for _ in range(2))
    want = [tuple(t.clone() for t in op.cost_grad(x, y, prm)) for x, y in ((xa, ya), (xb, yb))]
    ga, gb = torch.empty_like(xa), torch.empty_like(xb)
    ca, cb = (torch.empty(3, dtype=torch.float64, device="cuda") for _ in range(2))

    def eager(which):
        x, y, g, c = ((xa, ya, ga, ca), (xb, yb, gb, cb))[which]
        g.zero_()
        c.zero_()
        op.cost_grad(x, y, prm, g=g, cost=c)
        torch.cuda.synchronize()
        assert torch.equal(g, want[which][1]) and torch.equal(c[:1], want[which][0][:1])

    eager(0)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, capture_error_mode="thread_local"):
        op.cost_grad(xb, yb, prm, g=gb, cost=cb)
    eager(1)          # the captured call has not run yet
    eager(0)
    for _ in range(3):
        gb.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(gb, want[1][1]) and torch.equal(cb[:1], want[1][0][:1])
        eager(0)      # the replay has left the captured call's views behind
    op.close()
    ctx.close()
