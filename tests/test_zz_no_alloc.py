"""ddwc_dslash_apply_noalloc: the Dslash with its internal field in the library's static device
scratch instead of the context's workspace, for callers that cannot allocate.  Through the C ABI it
must give exactly (bit for bit) what ddwc_dslash_apply gives, on two calls in a row with the second
smaller than the first (the scratch keeps the first call's contents), in FP64 and FP32 on an
RHS-innermost and an RHS-major batch, and it takes the largest batch that fits and refuses a call whose field exceeds the scratch before
launching anything.  The FP64 result is also checked against the oracle (<= 1e-12 relative).
"""
import ctypes
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1211_1214_amd as dd  # noqa: E402
from oracle import dirac  # noqa: E402
from oracle.schwarz import Schwarz  # noqa: E402
from paper_1211_1214_amd import binding, inputs  # noqa: E402

pytestmark = pytest.mark.gpu
LAT, BLK = (8, 4, 4, 4), (2, 2, 2, 2)
KAPPA = 0.121


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def noalloc(ctx, inp, out, nrhs, prec):
    return binding.lib().ddwc_dslash_apply_noalloc(ctx._h, ctypes.c_double(KAPPA), ctypes.c_void_p(inp.data_ptr()),
                                                   ctypes.c_void_p(out.data_ptr()), int(nrhs), int(prec),
                                                   binding._stream())


@pytest.fixture(scope="module")
def env():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    U = inputs.make_links(LAT, 0.3, 71)
    ctx = dd.Context(torch.from_numpy(U).to(dev), LAT, BLK, -1, 1.0)
    yield dev, U, ctx
    ctx.close()


@pytest.mark.parametrize("prec", [dd.FP64, dd.MIXED32])
def test_noalloc_matches_dslash_apply(env, prec):
    dev, U, ctx = env
    S = Schwarz(U, LAT, BLK, 1.0)
    D = S.D(dirac.mass(KAPPA))
    for nrhs in (5, 1):  # the second call is smaller than the first
        say("noalloc", prec, nrhs)
        psi = inputs.make_spinor(LAT, 72 + nrhs, nrhs=nrhs)
        inp = torch.from_numpy(psi.reshape(nrhs, -1, 4, 3)).to(dev)
        want = ctx.dslash_apply(KAPPA, inp, prec=prec)
        got = torch.full_like(inp, float("nan"))
        assert noalloc(ctx, inp, got, nrhs, prec) == binding.OK
        torch.cuda.synchronize()
        assert torch.equal(got, want), "noalloc differs from ddwc_dslash_apply"
        if prec == dd.FP64:
            g = got.cpu().numpy()
            for j in range(nrhs):
                w = dirac.apply(D, psi.reshape(nrhs, -1, 4, 3)[j])
                assert np.abs(g[j] - w).max() <= 1e-12 * np.abs(w).max()


def test_noalloc_rejects_oversized_batch(env):
    dev, U, ctx = env
    V = int(np.prod(LAT))
    nrhs = (256 << 20) // (2 * V * 192) + 1  # an FP64 field just beyond the 128 MiB scratch
    dummy = torch.zeros(16, dtype=torch.complex128, device=dev)
    rc = binding.lib().ddwc_dslash_apply_noalloc(ctx._h, ctypes.c_double(KAPPA), ctypes.c_void_p(dummy.data_ptr()),
                                                 ctypes.c_void_p(dummy.data_ptr()), int(nrhs), dd.FP64,
                                                 binding._stream())
    assert rc == binding.EINVAL
    assert b"static scratch" in binding.lib().ddwc_last_error()


def test_noalloc_takes_the_largest_batch(env):
    dev, U, ctx = env
    V = int(np.prod(LAT))
    nrhs = (128 << 20) // (V * 192)  # (1365 RHS: the field ends 0.1 MB before the scratch does)
    say("noalloc", nrhs)
    psi = torch.from_numpy(inputs.make_spinor(LAT, 79, nrhs=3).reshape(3, V, 4, 3)).to(dev)
    inp = psi[torch.arange(nrhs, device=dev) % 3].contiguous()
    got = torch.full_like(inp, float("nan"))
    assert noalloc(ctx, inp, got, nrhs, dd.FP64) == binding.OK
    torch.cuda.synchronize()
    want = ctx.dslash_apply(KAPPA, psi)
    assert torch.equal(got, want[torch.arange(nrhs, device=dev) % 3])
