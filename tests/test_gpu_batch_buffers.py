"""The buffers that batches share go with their context: its device memory is
back after it is closed, and a batch on a later context equals the single
solves."""
import numpy as np
import pytest

from gpu_common import to_dev
from paper_2108_04315_amd import synth

pytestmark = pytest.mark.gpu


def _batch(misr, side, n):
    import torch
    ctx = misr.Context(0)
    rng = np.random.default_rng(side)
    ops, ys, xs, single = [], [], [], []
    for i in range(n):
        ops.append(misr.Operator(ctx, 2 * side, 2 * side, 2, synth.frame_shifts(2, 4, 0.05, i),
                                 synth.psf_taps(0.8)))
        ys.append(to_dev(rng.uniform(0, 1, (4, side, side))))
        xs.append(torch.empty((2 * side, 2 * side), device="cuda"))
        single.append(torch.empty_like(xs[-1]))
    prm = misr.default_params(n_iter=3, x_init=1)
    misr.scg_solve_batch(ops, ys, xs, [prm] * n, trace=False)
    for o, y, x in zip(ops, ys, single):
        o.scg_solve(y, x, prm, trace=False)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(xs, single))
    for o in ops:
        o.close()
    ctx.close()


def test_batch_buffers_go_with_their_context():
    import torch
    from paper_2108_04315_amd import misr
    _batch(misr, 24, 2)
    _batch(misr, 768, 2)   # (kernels loaded, torch's own blocks cached)
    _batch(misr, 24, 2)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    _batch(misr, 768, 2)   # 2 x 47 MB of solve buffers
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] >= before - (32 << 20)
    _batch(misr, 32, 3)
