"""Narrow tiles of small images against variant 0's tiles for 16-bit storage and
detector counts: adjoint and gradient bit for bit, the cost to the order of its
FP64 sums, a forward rounded to 16 bits to one unit in the last place."""
import numpy as np
import pytest

from gpu_common import to_dev
from paper_2108_04315_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store", ["float16", "bfloat16", "counts"])
@pytest.mark.parametrize("h,w,s,P", [(25, 17, 2, 7), (72, 147, 2, 9), (30, 70, 3, 7),
                                     (50, 64, 1, 7), (30, 41, 4, 7)])
def test_narrow_equals_wide(h, w, s, P, store):
    import torch
    from paper_2108_04315_amd import misr
    ctx = misr.Context(0)
    rng = np.random.default_rng(h + w)
    shifts = np.array([(0.0, 0.0), (0.45, -0.3), (-0.52, 0.5)])
    dt = torch.float32 if store == "counts" else getattr(torch, store)
    x = to_dev(rng.uniform(0, 1, (s * h, s * w)), dt)
    r = to_dev(rng.standard_normal((3, h, w)), dt)
    kw = {}
    if store == "counts":
        y = torch.from_numpy(rng.integers(0, 60000, (3, h, w)).astype(np.uint16)
                             .view(np.int16)).to("cuda")
        kw = dict(y_u16=1, y_scale=1.0 / 60000)
    else:
        y = to_dev(rng.uniform(0, 1, (3, h, w)), dt)
    out = []
    for wide in (False, True):
        op = misr.Operator(ctx, s * h, s * w, s, shifts, synth.psf_taps(P / 8.0, P))
        if wide:
            op.set_tile(0)
        cost, g = op.cost_grad(x, y, misr.default_params(**kw))
        out.append((op.forward(x), op.adjoint(r), g, cost))
        torch.cuda.synchronize()
        op.close()
    (fa, aa, ga, ca), (fb, ab, gb, cb) = out
    assert torch.equal(aa, ab) and torch.equal(ga, gb)
    assert torch.all((ca - cb).abs() <= 1e-12 * cb.abs())
    ulp = {"float16": 2.0 ** -10, "bfloat16": 2.0 ** -7, "counts": 0.0}[store]
    assert torch.all((fa.double() - fb.double()).abs() <= ulp * fb.double().abs() + 1e-7 * (ulp > 0))
    ctx.close()
