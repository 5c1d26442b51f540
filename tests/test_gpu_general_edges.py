"""The matrix-free general kernels at the edges of their branches, against
the FP64 oracle: one pixel past and one short of an LR tile and an HR tile,
images smaller than a tile, every scale and number of taps an LR pixel has
(matrix-core cells up to five, the position loop beyond and at scale 1), a
prior without smoothing, and a solve whose trial forms its residual on the
fly; and a batch of both forms and two scales (a launch each) that equals the
single solves bit for bit."""
import numpy as np
import pytest

import oracle
from gpu_common import TOL_OP, TOL_SCG, rel_l2, to_dev, to_np
from oracle import scg as oscg
from test_gpu_general import _f32, _geometry, _solve_problem, ctx, misr  # noqa: F401

pytestmark = pytest.mark.gpu

# H, W, s, K, P: LR tiles are 8 x 64 pixels, HR tiles 16 x 64
EDGES = [(2, 2, 2, 1, 3), (16, 128, 2, 2, 5), (18, 130, 2, 3, 7), (14, 126, 2, 2, 3),
         (34, 66, 2, 2, 11), (48, 195, 3, 2, 3), (51, 63, 3, 3, 5), (27, 198, 3, 2, 9),
         (36, 260, 4, 2, 5), (32, 60, 4, 2, 15), (17, 65, 1, 2, 3), (15, 63, 1, 3, 7),
         (20, 66, 2, 16, 5)]


@pytest.mark.parametrize("H,W,s,K,P", EDGES)
def test_edges_against_oracle(misr, ctx, H, W, s, K, P):  # noqa: F811
    import torch
    shifts, psf, warps = _geometry(H, W, s, K, P, "both", 5)
    op = misr.Operator(ctx, H, W, s, shifts, psf, warps=warps)
    assert op.sparse_width == (0, 0)
    rng = np.random.default_rng(H * 1000 + W)
    x = _f32(rng.uniform(0, 1, (H, W)))
    y_ref = oracle.forward(x, shifts, psf, s, warps=warps)
    assert rel_l2(to_np(op.forward(to_dev(x))), y_ref) <= TOL_OP
    r = _f32(rng.standard_normal(y_ref.shape))
    a_ref = oracle.adjoint(r, shifts, psf, s, H, W, warps=warps)
    assert rel_l2(to_np(op.adjoint(to_dev(r))), a_ref) <= TOL_OP
    yy = _f32(y_ref + 0.05 * rng.standard_normal(y_ref.shape))
    J, g_ref, _ = oracle.cost_grad(x, yy, shifts, psf, s, warps=warps)
    cost, g = op.cost_grad(to_dev(x), to_dev(yy), misr.default_params(n_iter=0))
    torch.cuda.synchronize()
    assert abs(cost.cpu().numpy()[0] - J) <= TOL_OP * J
    assert rel_l2(to_np(g), g_ref) <= TOL_OP
    op.close()


@pytest.mark.parametrize("H,W,s,K,P", [(42, 66, 3, 3, 5), (34, 130, 2, 2, 9), (20, 67, 1, 2, 5)])
def test_solve_edges_against_oracle(misr, ctx, H, W, s, K, P):  # noqa: F811
    shifts, psf, warps, y, x0 = _solve_problem(H, W, s, K, P, "both", 9)
    x_o, tr_o, _ = oscg.solve(y, shifts, psf, s, x0, 10, warps=warps)
    op = misr.Operator(ctx, H, W, s, shifts, psf, warps=warps)
    x = to_dev(x0)
    its, _ = op.scg_solve(to_dev(y), x, misr.default_params(n_iter=10))
    assert rel_l2(to_np(x), x_o) <= TOL_SCG
    assert [t["success"] for t in its] == [t["success"] for t in tr_o]
    op.close()


def test_batch_of_forms_and_scales_equals_singles(misr, ctx):  # noqa: F811
    import torch
    ops, frames, starts, single = [], [], [], []
    for q, (H, W, s, ell) in enumerate([(40, 66, 2, False), (40, 66, 2, True),
                                        (42, 63, 3, False), (20, 70, 1, False)]):
        shifts, psf, warps, y, x0 = _solve_problem(H, W, s, 2, 5, "both", 11 + q)
        ops.append(misr.Operator(ctx, H, W, s, shifts, psf, warps=warps, general_ell=ell))
        frames.append(to_dev(y))
        starts.append(to_dev(x0))
        x = starts[-1].clone()
        ops[-1].scg_solve(frames[-1], x, misr.default_params(n_iter=6))
        single.append(x)
    misr.scg_solve_batch(ops, frames, starts, [misr.default_params(n_iter=6)] * 4)
    torch.cuda.synchronize()
    for a, b in zip(starts, single):
        assert torch.equal(a, b)
    for op in ops:
        op.close()
