"""Block solves on blocks so large that the hop masks of the global-memory minimal-residual kernel do not fit the LDS
(above 40448 sites of a parity), and on the nearest smaller size of the same shape, which it takes.  The solutions
are put into the C oracle's block operator in FP64: ||b - D_k x|| <= tol ||b|| up to the rounding of that operator."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1211_1214_amd as dd  # noqa: E402
from oracle import cref, dirac  # noqa: E402
from paper_1211_1214_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = 1e-10


@pytest.mark.parametrize("blk", [(16, 16, 16, 18), (16, 16, 16, 20)])
def test_block_beyond_the_masks(blk):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert (np.prod(blk) // 2 > 40448) == (blk[3] == 20)
    lat = tuple(2 * b for b in blk)
    U = inputs.make_links(lat, 0.3, 51)
    b = inputs.make_spinor(lat, 52)
    ctx = dd.Context(torch.from_numpy(U).cuda(), lat, blk, -1, 1.0)
    R = cref.CRef(U, lat, blk, 1.0)
    for prec in (dd.MIXED32, dd.MIXED16):
        print("large block", blk, prec, flush=True)
        x, st = ctx.block_solve(dd.BLACK, 0.121, torch.from_numpy(b).cuda(), tol=TOL, prec=prec)
        x = x.cpu().numpy().reshape(-1, 4, 3)
        assert st["rel_residual"] <= TOL
        black = np.abs(x).max(axis=(1, 2)) > 0
        assert black.sum() == black.size // 2  # zero on the other colour, and nowhere else
        r = (b.reshape(-1, 4, 3) - R.block_apply(dd.BLACK, dirac.mass(0.121), x).reshape(-1, 4, 3))[black]
        # (per lattice: each block meets tol; the oracle's own rounding is 1e-16 times the condition number of one product)
        assert np.linalg.norm(r) <= 1.01 * TOL * np.linalg.norm(b.reshape(-1, 4, 3)[black])
    ctx.close()
    R.close()
