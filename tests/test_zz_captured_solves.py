"""Solves on a stream that the caller is capturing are refused, the first and a
repeated one alike, and touch neither their image nor the capture: what else is
captured replays, and the solves run as before afterwards."""
import numpy as np
import pytest

from gpu_common import to_dev
from paper_2108_04315_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("solved_before", [False, True])
def test_solves_refuse_a_capturing_stream(solved_before):
    import torch
    from paper_2108_04315_amd import misr
    ctx = misr.Context(0)
    rng = np.random.default_rng(4)
    h, w, s = 30, 41, 2
    op = misr.Operator(ctx, s * h, s * w, s, synth.frame_shifts(s, 4, 0.05, 3),
                       synth.psf_taps(0.8))
    ref_op = misr.Operator(ctx, s * h, s * w, s, synth.frame_shifts(s, 4, 0.05, 3),
                           synth.psf_taps(0.8))
    y, ya = (to_dev(rng.uniform(0, 1, (4, h, w))) for _ in range(2))
    x0 = to_dev(rng.uniform(0, 1, (s * h, s * w)))
    prm = misr.default_params(n_iter=4)
    want = x0.clone()
    ref_op.scg_solve(y, want, prm)
    if solved_before:
        for _ in range(2):
            misr.scg_solve_batch([op], [ya], [x0.clone()], [prm], trace=False)
            op.scg_solve(ya, x0.clone(), prm, trace=False)
    g, c = torch.zeros_like(x0), torch.zeros(3, dtype=torch.float64, device="cuda")
    g_ref = op.cost_grad(x0, y)[1].clone()
    xs = x0.clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="thread_local"):
        with pytest.raises(misr.MisrError):
            op.scg_solve(y, xs, prm, trace=False)
        with pytest.raises(misr.MisrError):
            misr.scg_solve_batch([op], [y], [xs], [prm], trace=False)
        op.cost_grad(x0, y, g=g, cost=c)
    torch.cuda.synchronize()
    assert torch.equal(xs, x0)
    for _ in range(2):
        g.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(g, g_ref) and torch.equal(xs, x0)
        for batch in (False, True):
            out = x0.clone()
            if batch:
                misr.scg_solve_batch([op], [y], [out], [prm], trace=False)
            else:
                op.scg_solve(y, out, prm, trace=False)
            torch.cuda.synchronize()
            assert torch.equal(out, want)
    del graph
    for o in (op, ref_op):
        o.close()
    ctx.close()
