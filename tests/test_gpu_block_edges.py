"""The Schwarz block solvers at the edges of their ranges, against the C oracle's block solves: block
parities of less than one wave, of a ragged last wave (idle lanes), of whole waves, the largest one
that the LDS-resident kernel takes (768 sites), the smallest beyond it, and the largest that keeps its
FP32 residual in LDS in the global-memory kernel and one beyond (8^4).  Tolerance as for every block
solve at tol 1e-12: 1e-9 relative (max norm)."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1211_1214_amd as dd  # noqa: E402
from oracle import cref, dirac  # noqa: E402
from paper_1211_1214_amd import binding, inputs  # noqa: E402

pytestmark = pytest.mark.gpu
_want = {}
BLOCKS = [(2, 2, 2, 2), (2, 6, 2, 2), (2, 4, 4, 6), (4, 4, 4, 4), (6, 6, 6, 6), (8, 8, 6, 4), (10, 8, 6, 4),
          (12, 8, 6, 4), (8, 8, 8, 8)]


@pytest.mark.parametrize("prec,kernel", [(dd.MIXED32, 0), (dd.MIXED32, 1), (dd.MIXED16, 1)])
@pytest.mark.parametrize("blk", BLOCKS)
def test_block_solver_edges(blk, prec, kernel):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("block edges", blk, prec, kernel, flush=True)
    sys.stdout.flush()
    dev = torch.device("cuda:0")
    lat = tuple(2 * b for b in blk)
    U = inputs.make_links(lat, 0.3, 21)
    ctx = dd.Context(torch.from_numpy(U).to(dev), lat, blk, -1, 1.0)
    R = cref.CRef(U, lat, blk, 1.0)
    ctx.set_option(binding.OPT_BLOCK_KERNEL, kernel)
    try:
        b = inputs.make_spinor(lat, 22, nrhs=3)
        b[1] *= 1e-3  # right-hand sides of other norms, and one that is zero
        b[2] = 0
        m = dirac.mass(0.121)
        for colour in (dd.BLACK, dd.WHITE) if kernel == 0 else (dd.WHITE,):
            x, st = ctx.block_solve(colour, 0.121, torch.from_numpy(b).to(dev), tol=1e-12, prec=prec)
            x = x.cpu().numpy()
            for j in (0, 1):
                key = (blk, colour, j)
                if key not in _want:
                    _want[key] = R.block_solve(colour, m, b[j], 1e-13).reshape(b[j].shape)
                want = _want[key]
                assert np.abs(x[j] - want).max() <= 1e-9 * np.abs(want).max()
            assert np.all(x[2] == 0) and st["rel_residual"] <= 1e-12
    finally:
        ctx.close()
        R.close()
