"""Images so wide that the rows one workgroup reads span 2^30 elements and more
(offsets that no longer fit 32 bits as bytes), against the FP64 oracle on narrow
column slabs: the columns of these warps move by less than two pixels, so a
slab's inner columns depend on the slab alone."""
import numpy as np
import pytest

import oracle
from gpu_common import TOL_OP, rel_l2

pytestmark = pytest.mark.gpu


def test_forward_rows_spanning_more_than_32_bits():
    import torch
    from paper_2108_04315_amd import misr
    # an LR tile of 8 rows reads 10 rows of the warped image, 4 apart: the tile
    # from row 8 spans 37 rows of 2^25 elements, all inside the image
    H, W, P = 46, 1 << 25, 3
    warp = np.array([[4.0, 0.0, -27.4, 0.0, 1.0, 0.3]])
    psf = np.array([0.25, 0.5, 0.25])
    ctx = misr.Context(0)
    op = misr.Operator(ctx, H, W, 1, np.zeros((1, 2)), psf, warps=warp)
    assert op.sparse_width == (0, 0)
    gen = torch.Generator(device="cuda").manual_seed(1)
    x = torch.empty((H, W), device="cuda").uniform_(0, 1, generator=gen)
    y = op.forward(x)
    torch.cuda.synchronize()
    for c0 in (1000, W // 2 - 77, W - 5000):
        c1, pad = c0 + 200, 4
        xs = x[:, c0:c1].double().cpu().numpy()
        ref = oracle.forward(xs, np.zeros((1, 2)), psf, 1, warps=warp)
        got = y[:, :, c0 + pad:c1 - pad].double().cpu().numpy()
        assert np.abs(ref[0, 8:16, pad:-pad]).max() > 0.1
        assert rel_l2(got, ref[:, :, pad:-pad]) <= TOL_OP
    op.close()
    ctx.close()
