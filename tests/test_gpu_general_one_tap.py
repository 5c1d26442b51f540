"""General operators without a blur (a 1-tap PSF: one tap an LR pixel, so the
adjoint forms its window position by position at every scale), against the FP64
oracle: several HR tiles per axis, windows that start at odd, even and negative
positions, rotated and shifted frames."""
import numpy as np
import pytest

import oracle
from gpu_common import TOL_OP, rel_l2, to_dev, to_np
from test_gpu_general import _f32, ctx, misr, rot_warp  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [(50, 134, 2), (48, 195, 3), (36, 260, 4), (33, 130, 1), (2, 2, 2)]


def _warps(H, W, angle):
    return np.stack([rot_warp(0.0, H, W, 1.0, -1.0), rot_warp(angle, H, W, -2.3, 0.4),
                     rot_warp(-angle, H, W, 0.6, 3.0)])


@pytest.mark.parametrize("angle", [0.0, 0.03])
@pytest.mark.parametrize("H,W,s", CASES)
def test_one_tap_against_oracle(misr, ctx, H, W, s, angle):  # noqa: F811
    import torch
    warps, shifts, psf = _warps(H, W, angle), np.zeros((3, 2)), np.ones(1)
    op = misr.Operator(ctx, H, W, s, shifts, psf, warps=warps)
    assert op.sparse_width == (0, 0)
    rng = np.random.default_rng(H + W)
    x = _f32(rng.uniform(0, 1, (H, W)))
    y_ref = oracle.forward(x, shifts, psf, s, warps=warps)
    assert rel_l2(to_np(op.forward(to_dev(x))), y_ref) <= TOL_OP
    r = _f32(rng.standard_normal(y_ref.shape))
    assert rel_l2(to_np(op.adjoint(to_dev(r))),
                  oracle.adjoint(r, shifts, psf, s, H, W, warps=warps)) <= TOL_OP
    yy = _f32(y_ref + 0.05 * rng.standard_normal(y_ref.shape))
    J, g_ref, _ = oracle.cost_grad(x, yy, shifts, psf, s, warps=warps)
    cost, g = op.cost_grad(to_dev(x), to_dev(yy), misr.default_params(n_iter=0))
    torch.cuda.synchronize()
    assert abs(cost.cpu().numpy()[0] - J) <= TOL_OP * J
    assert rel_l2(to_np(g), g_ref) <= TOL_OP
    op.close()
