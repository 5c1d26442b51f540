"""Band strips at the sizes where they can go wrong: images smaller than a
band (every weight row cut by an edge), exactly one tile, one LR pixel more
than a tile, and shifts of both signs whose bands reach past either edge;
forward, adjoint and cost + gradient against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from gpu_common import TOL_OP, rel_l2, to_dev, to_np
from paper_2108_04315_amd import synth

pytestmark = pytest.mark.gpu

# LR rows, LR columns, scale, PSF size
SIZES = [(1, 2, 2, 7), (3, 5, 2, 7), (24, 48, 2, 7), (25, 49, 2, 7), (49, 60, 2, 5), (2, 3, 3, 7),
         (16, 32, 3, 7), (17, 33, 3, 3), (51, 57, 1, 7), (12, 25, 4, 7), (40, 20, 2, 11)]


@pytest.fixture(scope="module")
def misr():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_2108_04315_amd import misr as m
    return m


@pytest.fixture(scope="module")
def ctx(misr):
    c = misr.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("h,w,s,P", SIZES)
def test_strips_match_oracle(misr, ctx, h, w, s, P):
    rng = np.random.default_rng(h * 100 + w)
    f32 = lambda a: np.asarray(a, np.float32).astype(np.float64)  # noqa: E731
    shifts = np.array([(0.0, 0.0), (0.37, -0.44), (-0.6, 0.21), (0.5, 0.5)])
    psf = synth.psf_taps(P / 7.0, P)
    x = f32(rng.uniform(0, 1, (s * h, s * w)))
    y = f32(rng.uniform(0, 1, (4, h, w)))
    op = misr.Operator(ctx, s * h, s * w, s, shifts, psf)
    for v in (0, 1):
        op.set_tile(v)
        assert rel_l2(to_np(op.forward(to_dev(x))), oracle.forward(x, shifts, psf, s)) <= TOL_OP
        assert rel_l2(to_np(op.adjoint(to_dev(y))),
                      oracle.adjoint(y, shifts, psf, s, s * h, s * w)) <= TOL_OP
        cost, g = op.cost_grad(to_dev(x), to_dev(y))
        J, g_ref, _ = oracle.cost_grad(x, y, shifts, psf, s)
        assert abs(to_np(cost)[0] - J) <= TOL_OP * J
        assert rel_l2(to_np(g), g_ref) <= TOL_OP
    op.close()
