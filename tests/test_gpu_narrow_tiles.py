"""Narrow tiles of small images against variant 0's tiles (set_tile(0)): the
operators, the gradient and a solve agree bit for bit (every pixel's sums are
rounded alike; only FP64 reductions are ordered differently, which a cost
bound of 1e-12 covers), at tile edges, ragged sizes and the largest image of
the rule; the reported shape stays the variant's."""
import numpy as np
import pytest

from gpu_common import to_dev
from paper_2108_04315_amd import synth

pytestmark = pytest.mark.gpu

# LR rows, LR columns, scale, PSF size, data norm
CASES = [(24, 16, 2, 7, 2), (25, 17, 2, 7, 1), (72, 147, 2, 7, 2), (335, 310, 2, 7, 2),
         (40, 61, 2, 11, 2), (30, 70, 3, 7, 2), (96, 130, 3, 5, 1), (50, 64, 1, 7, 2),
         (30, 41, 4, 7, 2)]


@pytest.mark.parametrize("h,w,s,P,p", CASES)
def test_narrow_equals_wide(h, w, s, P, p):
    import torch
    from paper_2108_04315_amd import misr
    ctx = misr.Context(0)
    rng = np.random.default_rng(h * 1000 + w)
    shifts = np.array([(0.0, 0.0), (0.45, -0.3), (-0.52, 0.5)])
    x = to_dev(rng.uniform(0, 1, (s * h, s * w)))
    y = to_dev(rng.uniform(0, 1, (3, h, w)))
    out = []
    for wide in (False, True):
        op = misr.Operator(ctx, s * h, s * w, s, shifts, synth.psf_taps(P / 8.0, P))
        shape = (op.tile, op.tile_variant)
        if wide:
            op.set_tile(0)
        assert (op.tile, op.tile_variant) == shape
        cost, g = op.cost_grad(x, y, misr.default_params(data_p=p))
        xs = torch.empty_like(x)
        op.scg_solve(y, xs, misr.default_params(n_iter=5, x_init=1, data_p=p))
        out.append((op.forward(x), op.adjoint(y), g, xs, cost))
        torch.cuda.synchronize()
        op.close()
    for a, b in zip(out[0][:4], out[1][:4]):
        assert torch.equal(a, b)
    assert torch.all((out[0][4] - out[1][4]).abs() <= 1e-12 * out[1][4].abs())
    ctx.close()
