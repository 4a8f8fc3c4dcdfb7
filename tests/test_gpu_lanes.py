"""The LDS-resident block solver with one, two and four lanes per site: the most sites that take four (16), the fewest
that do not, and 4^4 blocks in a launch small enough for two lanes and in one that takes one.  Against the C oracle's
block solves (1e-9 relative in the max norm at tol 1e-12, as for every block solve)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1211_1214_amd as dd  # noqa: E402
from oracle import cref, dirac  # noqa: E402
from paper_1211_1214_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blk,lat,nrhs", [((2, 2, 2, 4), (4, 4, 4, 8), 3), ((4, 2, 2, 2), (16, 8, 8, 8), 5),
                                          ((2, 2, 6, 2), (4, 4, 12, 4), 3), ((4, 4, 4, 4), (16, 8, 8, 8), 3),
                                          ((4, 4, 4, 4), (16, 8, 8, 8), 17), ((4, 4, 4, 2), (16, 16, 8, 8), 9)])
def test_lanes_per_site(blk, lat, nrhs):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("lanes", blk, lat, nrhs, flush=True)
    U = inputs.make_links(lat, 0.3, 25)
    ctx = dd.Context(torch.from_numpy(U).cuda(), lat, blk, -1, 1.0)
    R = cref.CRef(U, lat, blk, 1.0)
    b = inputs.make_spinor(lat, 26, nrhs=nrhs)
    b[1] = 0
    for colour in (dd.BLACK, dd.WHITE):
        x, st = ctx.block_solve(colour, 0.121, torch.from_numpy(b).cuda(), tol=1e-12, prec=dd.MIXED32)
        x = x.cpu().numpy()
        want = R.block_solve(colour, dirac.mass(0.121), b[nrhs - 1], 1e-13).reshape(b[0].shape)
        assert np.abs(x[nrhs - 1] - want).max() <= 1e-9 * np.abs(want).max()
        assert np.all(x[1] == 0) and st["rel_residual"] <= 1e-12
    ctx.close()
    R.close()
