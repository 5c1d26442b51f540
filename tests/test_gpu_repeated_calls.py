"""Calls that reuse what an operator or a batch keeps (plan arrays, captured
solves, buffers) with other frames, parameters and entry points in between:
every result equals, bit for bit, that of a fresh operator."""
import numpy as np
import pytest

from gpu_common import to_dev
from paper_2108_04315_amd import synth

pytestmark = pytest.mark.gpu


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


def _op(misr, ctx, h, w, s=2, seed=3):
    return misr.Operator(ctx, s * h, s * w, s, synth.frame_shifts(s, 4, 0.05, seed),
                         synth.psf_taps(0.8))


def _solve(misr, op, y, stream=None, **kw):
    import torch
    x = torch.empty((op.H, op.W), device="cuda")
    op.scg_solve(y, x, misr.default_params(x_init=1, **kw), trace=False, stream=stream)
    return x


@pytest.mark.parametrize("h,w", [(20, 33), (150, 170)])
def test_calls_interleaved_on_one_operator(misr, ctx, h, w):
    import torch
    rng = np.random.default_rng(h)
    ys = [to_dev(rng.uniform(0, 1, (4, h, w))) for _ in range(3)]
    xs = [to_dev(rng.uniform(0, 1, (2 * h, 2 * w))) for _ in range(3)]
    calls = [lambda o, i: _solve(misr, o, ys[i], n_iter=6),
             lambda o, i: o.cost_grad(xs[i], ys[i])[1],
             lambda o, i: o.forward(xs[i]),
             lambda o, i: _solve(misr, o, ys[i], n_iter=6, lambda_reg=0.05),
             lambda o, i: o.adjoint(ys[i]),
             lambda o, i: _solve(misr, o, ys[i], n_iter=3, tile_lr=64),
             lambda o, i: o.cost_grad(xs[i], ys[i], misr.default_params(data_p=1))[1]]
    op = _op(misr, ctx, h, w)
    order = [(c, i) for r in range(2) for i in range(3) for c in range(len(calls))]
    got = [(c, i, calls[c](op, i)) for c, i in order]
    torch.cuda.synchronize()
    for c in range(len(calls)):
        for i in range(3):
            fresh = _op(misr, ctx, h, w)
            ref = calls[c](fresh, i)
            torch.cuda.synchronize()
            for cc, ii, out in got:
                if (cc, ii) == (c, i):
                    assert torch.equal(out, ref), (c, i)
            fresh.close()
    # the status is the last solve's, whatever ran since
    assert op.scg_status()["n_passes"] == 3
    op.close()


def test_solves_on_several_streams(misr, ctx):
    """Operators on streams of their own, their solves in flight together."""
    import torch
    rng = np.random.default_rng(0)
    ops = [_op(misr, ctx, 40 + 8 * i, 56) for i in range(3)]
    ys = [to_dev(rng.uniform(0, 1, (4, o.H // 2, o.W // 2))) for o in ops]
    refs = [_solve(misr, o, y, n_iter=8) for o, y in zip(ops, ys)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in ops]
    for _ in range(3):
        outs = [_solve(misr, o, y, s, n_iter=8) for o, y, s in zip(ops, ys, streams)]
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, refs))
    for o in ops:
        o.close()


def test_batches_alternate(misr, ctx):
    """Batches of other operators, sizes and lengths in turn share the batch
    buffers (grown, kept and given back between them)."""
    import torch
    rng = np.random.default_rng(1)
    sets = []
    for sizes in ([(20, 24), (60, 50)], [(90, 80), (20, 24), (33, 41)], [(16, 16)]):
        ops = [_op(misr, ctx, h, w, seed=h) for h, w in sizes]
        sets.append((ops, [to_dev(rng.uniform(0, 1, (4, h, w))) for h, w in sizes]))
    refs = [[_solve(misr, o, y, n_iter=5) for o, y in zip(*st)] for st in sets]
    for k in (0, 1, 2, 1, 0, 2, 0):
        ops, ys = sets[k]
        xs = [torch.empty((o.H, o.W), device="cuda") for o in ops]
        misr.scg_solve_batch(ops, ys, xs, [misr.default_params(n_iter=5, x_init=1)] * len(ops),
                             trace=False)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(xs, refs[k]))
    for ops, _ in sets:
        for o in ops:
            o.close()
