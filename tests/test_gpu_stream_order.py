"""Calls on one operator from two streams in turn, ordered by events alone: what
one call leaves on the device for the next is there whichever stream it ran on,
and every result equals a fresh operator's bit for bit."""
import numpy as np
import pytest

from gpu_common import to_dev
from paper_2108_04315_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w", [(21, 34), (310, 290)])
def test_one_operator_on_two_streams(h, w):
    import torch
    from paper_2108_04315_amd import misr
    ctx = misr.Context(0)
    rng = np.random.default_rng(w)
    s = 2

    def make():
        return misr.Operator(ctx, s * h, s * w, s, synth.frame_shifts(s, 4, 0.05, 3),
                             synth.psf_taps(0.8))
    ys = [to_dev(rng.uniform(0, 1, (4, h, w))) for _ in range(2)]
    xs = [to_dev(rng.uniform(0, 1, (s * h, s * w))) for _ in range(2)]

    def solve(op, i, st):
        x = torch.empty_like(xs[i])
        op.scg_solve(ys[i], x, misr.default_params(n_iter=4, x_init=1), trace=False, stream=st)
        return x
    calls = [lambda op, i, st: op.forward(xs[i], stream=st),
             lambda op, i, st: op.cost_grad(xs[i], ys[i], stream=st)[1], solve,
             lambda op, i, st: op.adjoint(ys[i], stream=st),
             lambda op, i, st: op.cost_grad(xs[i], ys[i], misr.default_params(tile_lr=64),
                                            stream=st)[1]]
    ref = {}
    for c, call in enumerate(calls):
        for i in range(2):
            op = make()
            ref[c, i] = call(op, i, None)
            torch.cuda.synchronize()
            op.close()
    op = make()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got, last = [], torch.cuda.Event()
    last.record()
    order = [int(v) for v in rng.integers(0, 2 * len(calls), 40)]
    for n, v in enumerate(order):
        st = streams[(n * n // 3) % 2]
        st.wait_event(last)
        with torch.cuda.stream(st):
            got.append((v // 2, v % 2, calls[v // 2](op, v % 2, st)))
        last = torch.cuda.Event()
        last.record(st)
    torch.cuda.synchronize()
    for c, i, out in got:
        assert torch.equal(out, ref[c, i]), (c, i)
    op.close()
    ctx.close()
