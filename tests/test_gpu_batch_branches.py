"""A batch of solves of six launch classes (more than the graph has branches;
two of them hold two solves), replayed with other work and synchronisations
between: every replay equals the single solves bit for bit, on images, costs
and accept counts."""
import numpy as np
import pytest

from gpu_common import to_dev
from paper_2108_04315_amd import synth

pytestmark = pytest.mark.gpu

# LR rows, LR columns, scale, PSF size: classes by scale and band length
SOLVES = [(60, 70, 2, 7), (50, 64, 3, 7), (40, 130, 1, 7), (33, 41, 4, 7), (64, 48, 2, 11),
          (30, 45, 3, 3), (91, 35, 2, 7), (25, 52, 3, 7)]


def test_batch_of_many_classes_replayed():
    import torch
    from paper_2108_04315_amd import misr
    ctx = misr.Context(0)
    rng = np.random.default_rng(5)
    shifts = np.array([(0.0, 0.0), (0.45, -0.3), (-0.2, 0.5)])
    prm = [misr.default_params(n_iter=8 + i % 3, x_init=1) for i in range(len(SOLVES))]
    ops, ys = [], []
    for h, w, s, P in SOLVES:
        ops.append(misr.Operator(ctx, s * h, s * w, s, shifts, synth.psf_taps(P / 8.0, P)))
        ys.append(to_dev(rng.uniform(0, 1, (3, h, w))))
    for rep in range(4):
        xs = [torch.empty((s * h, s * w), device="cuda") for h, w, s, _ in SOLVES]
        misr.scg_solve_batch(ops, ys, xs, prm)
        if rep == 1:
            torch.cuda.synchronize()
        for op, y, x, p in zip(ops, ys, xs, prm):
            alone = torch.empty_like(x)
            its, _ = op.scg_solve(y, alone, p)
            assert torch.equal(alone, x), (rep, op.s)
            assert len(its) == p.n_iter
        ys = [torch.flip(y, (1,)).contiguous() for y in ys]   # new frames, new buffers
    for op in ops:
        op.close()
    ctx.close()
