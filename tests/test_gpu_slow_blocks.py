"""Block solves at masses where minimal residual converges slowly on some block, so that its kernel has to leave the
rest to BiCGStab: with one, two and four lanes per site and with the global-memory kernel (FP32 and FP16), at a tight
tolerance and at loose ones, where a residual starts close to its goal.  The same iteration is run here on the oracle's
block operator first and has to show such a block; the solutions are put into that operator (per lattice
||b - D_k x|| <= tol ||b||, as each block meets tol)."""
import numpy as np
import pytest
import scipy.sparse.linalg as sla

torch = pytest.importorskip("torch")

import paper_1211_1214_amd as dd  # noqa: E402
from oracle import dirac, lattice as lt  # noqa: E402
from oracle.schwarz import Schwarz  # noqa: E402
from paper_1211_1214_amd import binding, inputs  # noqa: E402

WINDOW, GAIN = 8, 0.16  # the kernels' rule: steps, and the least fall of ||r|| in them
CASES = [((2, 2, 2, 4), (4, 4, 4, 8), 0.25), ((4, 4, 4, 4), (8, 8, 8, 8), 0.18), ((6, 4, 4, 4), (12, 8, 8, 8), 0.17)]


class Blocks:
    """The black blocks' operator of one lattice, and minimal residual on its even part."""

    def __init__(self, blk, lat, kappa):
        S = Schwarz(inputs.make_links(lat, 0.3, 61), lat, blk, 1.0)
        n = lt.coords(lat) // np.array(blk)
        black = n.sum(axis=1) % 2 == 0
        even = lt.coords(lat).sum(axis=1) % 2 == 0
        dofs = lambda m: (12 * np.nonzero(m)[0][:, None] + np.arange(12)).ravel()  # noqa: E731
        self.black = dofs(black)
        D = S.D(dirac.mass(kappa)).tocsr()
        D = D[self.black][:, self.black]  # black blocks do not touch: the blocks' operators
        e, o = np.nonzero(np.repeat(even[black], 12))[0], np.nonzero(np.repeat(~even[black], 12))[0]
        self.D, self.e, self.o = D, e, o
        self.ee, self.eo, self.oe = D[e][:, e], D[e][:, o], D[o][:, e]
        self.oo = sla.splu(D[o][:, o].tocsc())
        rank = np.ravel_multi_index(n.T, np.array(lat) // np.array(blk))
        self.block = np.unique(np.repeat(rank[black], 12)[e], return_inverse=True)[1]
        self.blocks = np.unique(np.repeat(rank[black], 12), return_inverse=True)[1]

    def slow(self, b, tol):
        """Whether some block's ||r|| falls by less than GAIN (with a margin) in WINDOW steps before it is at tol / 4."""
        nrm = lambda v, k: np.sqrt(np.bincount(k, np.abs(v) ** 2))  # noqa: E731
        b = b.reshape(-1)[self.black]
        goal = 0.25 * tol * nrm(b, self.blocks)
        r = b[self.e] - self.eo @ self.oo.solve(b[self.o])
        window = nrm(r, self.block)
        for it in range(1, 5 * WINDOW + 1):
            t = self.ee @ r - self.eo @ self.oo.solve(self.oe @ r)
            dot = lambda u, v: np.bincount(self.block, (u.conj() * v).real) + 1j * np.bincount(self.block, (u.conj() * v).imag)  # noqa: E731
            r = r - (dot(t, r) / dot(t, t))[self.block] * t
            if it % WINDOW == 0:
                now = nrm(r, self.block)
                if np.any((now > 1.25 * GAIN * window) & (now > 1.5 * goal)):
                    return True
                window = now
        return False


_cache = {}


def blocks(case):
    if case not in _cache:
        _cache[case] = Blocks(*case)
    return _cache[case]


@pytest.mark.parametrize("case", CASES)
def test_minimal_residual_is_slow_there(case):
    b = inputs.make_spinor(case[1], 62, nrhs=3)
    for tol in (1e-1, 1e-2, 1e-10):
        assert any(blocks(case).slow(b[j], tol) for j in range(3))


@pytest.mark.gpu
@pytest.mark.parametrize("prec,kernel", [(dd.MIXED32, 0), (dd.MIXED32, 1), (dd.MIXED16, 1)])
@pytest.mark.parametrize("case", CASES)
def test_slow_blocks(case, prec, kernel):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    blk, lat, kappa = case
    B = blocks(case)
    ctx = dd.Context(torch.from_numpy(inputs.make_links(lat, 0.3, 61)).cuda(), lat, blk, -1, 1.0)
    ctx.set_option(binding.OPT_BLOCK_KERNEL, kernel)
    b = inputs.make_spinor(lat, 62, nrhs=3)
    for tol in (1e-1, 1e-2, 1e-10):
        print("slow blocks", blk, prec, kernel, tol, flush=True)
        x, st = ctx.block_solve(dd.BLACK, kappa, torch.from_numpy(b).cuda(), tol=tol, prec=prec)
        assert st["rel_residual"] <= tol and st["outer_iters"] >= 2
        x = x.cpu().numpy().reshape(3, -1)
        for j in range(3):
            w = b[j].reshape(-1)[B.black]
            assert np.linalg.norm(w - B.D @ x[j][B.black]) <= 1.01 * tol * np.linalg.norm(w)
    ctx.close()
