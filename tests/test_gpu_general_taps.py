"""Every PSF size of the matrix-free general operators at every scale (each has
its own unrolling of the forward's window sums; the adjoint forms its window by
cells or position by position, with 1 to 15 taps an LR pixel), against the FP64
oracle on images of several tiles with ragged edges."""
import numpy as np
import pytest

import oracle
from gpu_common import TOL_OP, rel_l2, to_dev, to_np
from test_gpu_general import _f32, _geometry, ctx, misr  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [1, 3, 5, 7, 9, 11, 13, 15])
@pytest.mark.parametrize("s,H,W", [(1, 19, 131), (2, 38, 134), (3, 51, 201), (4, 36, 264)])
def test_every_psf_size(misr, ctx, s, H, W, P):  # noqa: F811
    shifts, psf, warps = _geometry(H, W, s, 2, P, "both", P)
    op = misr.Operator(ctx, H, W, s, shifts, psf, warps=warps)
    assert op.sparse_width == (0, 0)
    rng = np.random.default_rng(s * 100 + P)
    x = _f32(rng.uniform(0, 1, (H, W)))
    y_ref = oracle.forward(x, shifts, psf, s, warps=warps)
    assert rel_l2(to_np(op.forward(to_dev(x))), y_ref) <= TOL_OP
    r = _f32(rng.standard_normal(y_ref.shape))
    assert rel_l2(to_np(op.adjoint(to_dev(r))),
                  oracle.adjoint(r, shifts, psf, s, H, W, warps=warps)) <= TOL_OP
    yy = _f32(y_ref + 0.05 * rng.standard_normal(y_ref.shape))
    J, g_ref, _ = oracle.cost_grad(x, yy, shifts, psf, s, warps=warps)
    cost, g = op.cost_grad(to_dev(x), to_dev(yy), misr.default_params(n_iter=0))
    assert abs(to_np(cost)[0] - J) <= TOL_OP * J
    assert rel_l2(to_np(g), g_ref) <= TOL_OP
    op.close()
