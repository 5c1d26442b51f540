"""Narrow tiles at the image's right edge where their width does not divide the
wide tile's (bands of 10 to 16 at scale 2, of up to 8 at scale 1): tiles that lie
across two wide ones, the second of them cut by the edge.  Cost and gradient
against the FP64 oracle, and the gradient against the wide tiles' to the rounding
of its FP32 sums."""
import numpy as np
import pytest

import oracle
from gpu_common import TOL_OP, rel_l2, to_dev, to_np
from paper_2108_04315_amd import synth

pytestmark = pytest.mark.gpu

# LR rows, LR columns, scale, PSF size: HR columns 242 to 254 (scale 2), 114 to 119
CASES = [(60, 121, 2, 9), (60, 124, 2, 11), (50, 127, 2, 13), (60, 128, 2, 9), (130, 114, 1, 3),
         (130, 117, 1, 5), (110, 119, 1, 7), (130, 120, 1, 5), (60, 283, 2, 11), (60, 137, 2, 11)]


@pytest.mark.parametrize("h,w,s,P", CASES)
def test_tiles_across_two_wide_ones(h, w, s, P):
    import torch
    from paper_2108_04315_amd import misr
    ctx = misr.Context(0)
    H, W = s * h, s * w
    shifts = np.array([(0.0, 0.0), (0.45, -0.3)])
    psf = synth.psf_taps(P / 8.0, P)
    rng = np.random.default_rng(h + w)
    x = np.float32(rng.uniform(0, 1, (H, W))).astype(np.float64)
    y = np.float32(rng.uniform(0, 1, (2, h, w))).astype(np.float64)
    J, g_ref, _ = oracle.cost_grad(x, y, shifts, psf, s)
    out = []
    for wide in (False, True):
        op = misr.Operator(ctx, H, W, s, shifts, psf)
        if wide:
            op.set_tile(0)
        cost, g = op.cost_grad(to_dev(x), to_dev(y))
        torch.cuda.synchronize()
        assert abs(to_np(cost)[0] - J) <= TOL_OP * J
        assert rel_l2(to_np(g), g_ref) <= TOL_OP
        assert np.abs(to_np(g) - g_ref).max() <= TOL_OP * np.abs(g_ref).max()
        out.append(g)
        op.close()
    assert (out[0] - out[1]).abs().max() <= 1e-6 * out[1].abs().max()
    ctx.close()
