"""Global solves of lattices whose parity fits the LDS-resident solver (up to 768 sites): the smallest, one that does
not fill its last wavefront's workgroup, the largest, and the first beyond it; both time boundary conditions; one,
some and a zero right-hand side; and a kappa where minimal residual is left for BiCGStab, at tight and at loose tolerances.  Against the C oracle's
solves (1e-9 relative in the max norm at tol 1e-12, as for every solve)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1211_1214_amd as dd  # noqa: E402
from oracle import cref, dirac  # noqa: E402
from paper_1211_1214_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu
LATTICES = [((4, 4, 4, 4), (2, 2, 2, 2)), ((4, 12, 4, 4), (2, 2, 2, 2)), ((12, 8, 4, 4), (6, 4, 2, 2)),
            ((8, 8, 8, 4), (4, 4, 4, 2))]


@pytest.mark.parametrize("prec", [dd.MIXED32, dd.MIXED16])
@pytest.mark.parametrize("bc", [-1, 1])
@pytest.mark.parametrize("lat,blk", LATTICES)
def test_resident_solve(lat, blk, bc, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U = inputs.make_links(lat, 0.3, 33)
    ctx = dd.Context(torch.from_numpy(U).cuda(), lat, blk, bc, 1.0)
    R = cref.CRef(U, lat, blk, 1.0, bc)
    b = inputs.make_spinor(lat, 34, nrhs=5)
    b[1] = 0
    b[3] *= 1e-3
    # (0.133 is so close to critical on 12x8x4x4, 1000 iterations and more, and beyond it on periodic lattices, that the
    # oracle's own solve does not always converge there: 85 iterations at 0.126)
    slow = () if bc > 0 else ((0.128 if lat == (12, 8, 4, 4) else 0.133, 5),)
    for kappa, nrhs in ((0.121, 5), (0.121, 1)) + slow:
        print("resident", lat, bc, prec, kappa, nrhs, flush=True)
        x, st = ctx.solve(kappa, torch.from_numpy(b[:nrhs].copy()).cuda(), tol=1e-12, prec=prec)
        print(st, flush=True)
        x = x.cpu().numpy().reshape(nrhs, -1)
        assert st["rel_residual"] <= 1e-12 and st["inner_iters"] > 0
        # (two launches of the resident solver reach 1e-12 from its floor of 2e-6: a third outer step is the change-over)
        assert kappa == 0.121 or st["outer_iters"] >= 3
        for j in {0, nrhs - 1, nrhs // 2 + 1} - {1}:
            if j < nrhs:
                w = R.solve(dirac.mass(kappa), b[j], 1e-13).reshape(-1)
                assert np.abs(x[j] - w).max() <= 1e-9 * np.abs(w).max()
        assert nrhs == 1 or np.all(x[1] == 0)
    # at loose tolerances a residual starts close to its goal
    for tol in (1e-1, 1e-2):
        for kappa, nrhs in slow:
            x, st = ctx.solve(kappa, torch.from_numpy(b[:nrhs].copy()).cuda(), tol=tol, prec=prec)
            x = x.cpu().numpy()
            assert st["rel_residual"] <= tol
            for j in (0, nrhs - 1):
                r = b[j].reshape(-1) - R.dslash(dirac.mass(kappa), x[j]).reshape(-1)
                assert np.linalg.norm(r) <= 1.01 * tol * np.linalg.norm(b[j])
    # an iteration limit is refused as before
    with pytest.raises(dd.binding.DDWCError):
        ctx.solve(0.121, torch.from_numpy(b).cuda(), tol=1e-12, maxit=2, prec=prec)
    ctx.close()
