"""Dispatch orders of the operator: the first call of a shape (its table is written on the call's stream), later ones, one on
another stream, and one that is captured into a graph before its table exists give what index order gives
(ddwc_dslash_apply_noalloc), bit for bit; and so does a solve."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1211_1214_amd as dd  # noqa: E402
from paper_1211_1214_amd import binding, inputs  # noqa: E402

pytestmark = pytest.mark.gpu
KAPPA = 0.121


@pytest.fixture(autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def context(lat, blk):
    return dd.Context(torch.from_numpy(inputs.make_links(lat, 0.3, 81)).cuda(), lat, blk, -1, 1.0)


def spinors(lat, nrhs):
    return torch.from_numpy(inputs.make_spinor(lat, 82, nrhs=nrhs)).cuda()


def index_order(ctx, v, prec):
    out = torch.full_like(v, float("nan"))
    assert binding.lib().ddwc_dslash_apply_noalloc(ctx._h, KAPPA, v.data_ptr(), out.data_ptr(), v.shape[0], int(prec),
                                                   binding._stream()) == binding.OK
    return out


@pytest.mark.parametrize("lat,blk", [((24, 12, 12, 12), (6, 6, 6, 6)), ((36, 8, 16, 8), (6, 2, 4, 4)),
                                     ((16, 16, 12, 12), (2, 2, 2, 2))])
@pytest.mark.parametrize("prec", [dd.FP64, dd.MIXED32])
def test_first_call(lat, blk, prec):
    ctx = context(lat, blk)
    for nrhs in (1, 5, 9):
        print("tile order", lat, blk, prec, nrhs, flush=True)
        v = spinors(lat, nrhs)
        want = index_order(ctx, v, prec)
        for _ in range(2):
            assert torch.equal(ctx.dslash_apply(KAPPA, v, prec=prec), want)
    ctx.close()


def test_other_stream():
    lat, blk = (16, 16, 16, 16), (4, 4, 4, 4)  # (the two precisions share a table here, and no other memory)
    ctx = context(lat, blk)
    v = spinors(lat, 1)
    want = index_order(ctx, v, dd.FP64), index_order(ctx, v, dd.MIXED32)
    outs = torch.empty_like(v), torch.empty_like(v)
    streams = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for s, o, prec in zip(streams, outs, (dd.FP64, dd.MIXED32)):
        with torch.cuda.stream(s):
            ctx.dslash_apply(KAPPA, v, out=o, prec=prec)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], want[0]) and torch.equal(outs[1], want[1])
    ctx.close()


@pytest.mark.parametrize("warm", [False, True])
def test_captured_call(warm):
    lat, blk = (24, 12, 12, 12), (6, 6, 6, 6)
    ctx = context(lat, blk)
    v = spinors(lat, 3)
    ctx.dslash_apply(KAPPA, v)  # the workspace, but not the table of one right-hand side
    w, out = v[:1].clone(), torch.empty_like(v[:1])
    if warm:
        ctx.dslash_apply(KAPPA, w, out=out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.dslash_apply(KAPPA, w, out=out)
    for k in range(4):
        w.copy_(v[k % 3:k % 3 + 1])
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, index_order(ctx, w, dd.FP64))
        assert torch.equal(out, ctx.dslash_apply(KAPPA, w))
    del g
    ctx.close()


@pytest.mark.parametrize("prec", [dd.FP64, dd.MIXED32])
@pytest.mark.parametrize("lat,blk", [((24, 16, 16, 16), (4, 4, 4, 4)), ((28, 16, 16, 16), (2, 4, 4, 4))])
def test_solve(lat, blk, prec):
    """One right-hand side below and from the size on from which the global solver's tiles are ordered: the same bits."""
    ctx = context(lat, blk)
    v = spinors(lat, 1)
    x, _ = ctx.solve(KAPPA, v, tol=1e-10, prec=prec)
    ctx.set_option(binding.OPT_TILE_ORDER, 0)
    y, _ = ctx.solve(KAPPA, v, tol=1e-10, prec=prec)
    assert torch.equal(x, y)
    ctx.close()
