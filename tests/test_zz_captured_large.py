"""Calls captured into the caller's own graphs on images of several hundred
tiles, whose work lists are copied from host memory at every replay, with eager
calls between the replays that rebuild those lists, outgrow the operator's
arrays and replace its tile buffers (another tile size, another tile variant, a
solve): every replay equals the eager call bit for bit."""
import numpy as np
import pytest

from gpu_common import to_dev
from paper_2108_04315_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,s", [(700, 650, 2), (430, 500, 3)])
def test_replays_between_eager_calls(h, w, s):
    import torch
    from paper_2108_04315_amd import misr
    ctx = misr.Context(0)
    rng = np.random.default_rng(h)
    shifts = np.array([(0.0, 0.0), (0.45, -0.3), (-0.2, 0.4)])
    op = misr.Operator(ctx, s * h, s * w, s, shifts, synth.psf_taps(0.8, 7))
    x = to_dev(rng.uniform(0, 1, (s * h, s * w)))
    y = to_dev(rng.uniform(0, 1, (3, h, w)))
    plain, tiled = misr.default_params(), misr.default_params(tile_lr=200)
    outs = [torch.zeros_like(y)] + [torch.zeros_like(x) for _ in range(3)]
    costs = [torch.zeros(3, dtype=torch.float64, device="cuda") for _ in range(2)]
    calls = [lambda: op.forward(x, outs[0]), lambda: op.adjoint(y, outs[1]),
             lambda: op.cost_grad(x, y, plain, g=outs[2], cost=costs[0]),
             lambda: op.cost_grad(x, y, tiled, g=outs[3], cost=costs[1])]

    def eager():
        for c in calls:
            c()
        torch.cuda.synchronize()
        return [t.clone() for t in outs + costs]

    want = eager()
    graphs = []
    for c in calls:
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1], capture_error_mode="thread_local"):
            c()

    def disturb(n):
        """Other lists, more and larger arrays, other buffers."""
        xs = torch.empty_like(x)
        op.scg_solve(y, xs, misr.default_params(n_iter=2, x_init=1, tile_lr=(64, 32, 100)[n]))
        op.set_tile(1)
        op.cost_grad(x, y, misr.default_params(data_p=1))
        op.scg_solve(y, xs, misr.default_params(n_iter=2, x_init=1))
        op.set_tile(0)
        torch.cuda.synchronize()

    for n in range(3):
        disturb(n)
        junk = [torch.full_like(x, 7.0) for _ in range(4)]   # over whatever was freed
        torch.cuda.synchronize()
        for order in (range(4), reversed(range(4))):
            for t in outs + costs:
                t.zero_()
            for i in order:
                graphs[i].replay()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(outs + costs, want))
        del junk
        got = eager()   # and the eager calls find what they need
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    del graphs
    op.close()
    ctx.close()
