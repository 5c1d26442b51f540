"""The SCG steps at the end of a pass (run by the last workgroup of a solve to
finish) over the numbers of workgroups where their sums change shape: one,
one row per summing thread and one more, four rows per thread and one more,
and the tiles of a tiled solve, which share one count.  A solve's final cost
is the cost at its result as evaluated alone (the same FP32 sums per pixel,
so FP64 sums apart by their order only, at an iterate rounded once more:
1e-6), every pass runs its steps exactly once (pass numbers and accept
counts), and a repetition gives the same bits."""
import numpy as np
import pytest

from gpu_common import to_dev
from paper_2108_04315_amd import synth

pytestmark = pytest.mark.gpu

# LR rows, LR columns, tile (0: untiled); at scale 2 a narrow tile covers
# 24 x 16 LR pixels and a wide one 24 x 48
CASES = [(8, 8, 0), (24, 16 * 256, 0), (24, 16 * 257, 0), (24 * 32, 48 * 32, 0),
         (24 * 41, 48 * 25, 0), (130, 210, 64)]


@pytest.mark.parametrize("h,w,tile", CASES)
def test_steps_once_per_pass(h, w, tile):
    import torch
    from paper_2108_04315_amd import misr
    ctx = misr.Context(0)
    rng = np.random.default_rng(h + w)
    shifts = np.array([(0.0, 0.0), (0.45, -0.3)])
    op = misr.Operator(ctx, 2 * h, 2 * w, 2, shifts, synth.psf_taps(0.8, 7))
    y = to_dev(rng.uniform(0, 1, (2, h, w)))
    prm = misr.default_params(n_iter=12, x_init=1, tile_lr=tile)
    runs = []
    for _ in range(2):
        x = torch.empty((2 * h, 2 * w), device="cuda")
        its, info = op.scg_solve(y, x, prm)
        runs.append((x, [t["E"] for t in its], info))
    (x, costs, info), (x2, costs2, info2) = runs
    assert torch.equal(x, x2) and costs == costs2 and info == info2
    assert len(costs) == 12 and 0 < info["n_success"] <= 12
    assert all(b <= a for a, b in zip(costs, costs[1:]))
    cost, _ = op.cost_grad(x, y, misr.default_params())
    assert abs(cost.cpu().numpy()[0] - costs[-1]) <= 1e-6 * costs[-1]
    op.close()
    ctx.close()
