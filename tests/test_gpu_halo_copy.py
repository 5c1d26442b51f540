"""Halo copies at the sizes where their chunks can go wrong: strips narrower
and longer than one workgroup's share, corner rectangles of a single pixel and
ragged last tiles; the tiled gradient equals the untiled one bit for bit (the
same sums per pixel), the tiled solve the untiled one to FP32 rounding of its
differently ordered FP64 reductions (none seen by a short solve)."""
import numpy as np
import pytest

from gpu_common import to_dev
from paper_2108_04315_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,tile,halo", [(70, 45, 32, 8), (33, 300, 32, 4), (1100, 40, 36, 5),
                                           (64, 65, 64, 8)])
def test_tiled_solve_equals_untiled(h, w, tile, halo):
    import torch
    from paper_2108_04315_amd import misr
    ctx = misr.Context(0)
    s = 2
    op = misr.Operator(ctx, s * h, s * w, s, synth.frame_shifts(s, 4, 0.05, 3),
                       synth.psf_taps(0.8))
    rng = np.random.default_rng(h + w)
    y = to_dev(rng.uniform(0, 1, (4, h, w)))
    out = []
    for t in (0, tile):
        x = torch.empty((s * h, s * w), device="cuda")
        op.scg_solve(y, x, misr.default_params(n_iter=6, x_init=1, tile_lr=t, halo_lr=halo))
        out.append(x.double())
    err = float((out[0] - out[1]).norm() / out[0].norm())
    assert err <= 1e-6, err
    op.close()
    ctx.close()
