"""The calls a user of the library makes, as measurable cases: sizes, inputs, one pass, its work and
what it returns in plain 64-bit arithmetic.

The range is the library's own: the smallest lattices (4x4^3) to the largest (64x32^3), one
right-hand side to a whole batch of noise vectors, the operator alone, the Schwarz block solves, the
global solve, and whole estimates (global Schur factor, nested decomposition, gradient), in FP64 and
in the mixed FP32 and FP16 precisions, with even blocks and with odd (ragged) ones.
"""
import math

import numpy as np
import torch

import paper_1211_1214_amd as dd
from paper_1211_1214_amd import autograd

CSW, EPS = 1.0, 0.3  # clover coefficient and disorder of the synthetic links
PREC = {"fp64": dd.FP64, "mixed32": dd.MIXED32, "mixed16": dd.MIXED16}


def _case(name, op, lat, blk, nrhs, prec, **more):
    c = {"op": op, "lat": lat, "blk": blk, "nrhs": nrhs, "prec": prec, "kappa1": 0.1200, "kappa2": 0.1205, "tol": 1e-10}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the operator on the smallest lattice: launches and latency, as in a test or a tight loop
        _case("dslash 4x4^3 fp64", "dslash", "4x4x4x4", "2x2x2x2", 1, "fp64"),
        # the operator on one field of the 48x24^3 workload, as an outer solver or a measurement calls it
        _case("dslash 48x24^3 fp64", "dslash", "48x24x24x24", "6x6x6x6", 1, "fp64"),
        # the operator in FP32 on that workload's whole batch of noise vectors
        _case("dslash 48x24^3 x12", "dslash", "48x24x24x24", "6x6x6x6", 12, "mixed32"),
        # all Schwarz blocks of one colour, whole batch (the a3 step of every estimate)
        _case("block solve 48x24^3 x12", "block_solve", "48x24x24x24", "6x6x6x6", 12, "mixed32"),
        # the global solve of the batch
        _case("solve 48x24^3 x12", "solve", "48x24x24x24", "6x6x6x6", 12, "mixed32"),
        # one propagator-like solve entirely in FP64
        _case("solve 32x16^3 fp64", "solve", "32x16x16x16", "4x4x4x4", 1, "fp64"),
        # odd block extents, a handful of right-hand sides
        _case("solve 24x12^3 odd x5", "solve", "24x12x12x12", "3x3x3x3", 5, "mixed32"),
        # the smallest whole estimate: nothing but launches and waits
        _case("estimate 4x4^3 x8", "estimate", "4x4x4x4", "2x2x2x2", 8, "mixed32", kappa2=0.1210),
        # the reweighting factor of one 48x24^3 configuration, 12 noise vectors
        _case("estimate 48x24^3 x12", "estimate", "48x24x24x24", "6x6x6x6", 12, "mixed32"),
        # the largest lattice with 8^4 blocks, FP16 storage in the inner solves
        _case("estimate 64x32^3 fp16 x6", "estimate", "64x32x32x32", "8x8x8x8", 6, "mixed16"),
        # forward and backward of log W_gl in kappa2 and the links, as in reweighting-aware HMC
        _case("gradient 32x16^3 x8", "gradient", "32x16x16x16", "4x4x4x4", 8, "mixed32"),
        # the nested factor of one colour's 8^4 blocks split again into 4^4 blocks
        _case("nested 32x16^3 x8", "nested", "32x16x16x16", "8x8x8x8", 8, "mixed32", inner="4x4x4x4"),
    ]


def draw(rng):
    """One more case: the operation, precision, block shape and batch of a user's program, with the
    number of (site, right-hand side) pairs spread over the logarithm of the whole range."""
    op = rng.choice(["dslash", "dslash", "block_solve", "solve", "solve", "estimate", "estimate", "gradient", "nested"])
    prec = rng.choice(["fp64", "mixed32", "mixed32", "mixed16"] if op in ("solve", "estimate") else ["fp64", "mixed32", "mixed32"])
    most = {"dslash": 8e6, "block_solve": 8e6, "solve": 8e6, "estimate": 8e6, "gradient": 1e6, "nested": 1e6}[op]
    if prec == "fp64":
        most /= 8  # FP64 takes several times as long
    pairs = math.exp(rng.uniform(math.log(2e3), math.log(most)))
    odd = op in ("dslash", "solve") and prec != "mixed16" and rng.random() < 0.25
    if odd:
        pairs = min(pairs, 3e5)
    b = rng.choice([3, 5] if odd else [8] if op == "nested" else [2, 4, 4, 6, 8])
    blk = [b] * 4
    if op != "nested" and rng.random() < 0.4:  # anisotropic blocks
        blk[rng.randrange(4)] = rng.choice([2, 3, 4] if odd else [2, 4, 6])
    n = [2 * v for v in blk]
    nrhs = rng.choice([1, 1, 2, 3, 4, 5, 7, 8, 9, 12, 13, 16])
    while math.prod(n) * nrhs > most and nrhs > 1:
        nrhs -= 1
    while True:  # grow a random direction by two blocks while the pairs allow it
        grow = [m for m in range(4) if math.prod(n) // n[m] * (n[m] + 2 * blk[m]) * nrhs <= pairs and n[m] + 2 * blk[m] <= 64]
        if not grow:
            break
        m = rng.choice(grow)
        n[m] += 2 * blk[m]
    text = lambda v: "x".join(str(x) for x in v)  # noqa: E731
    more = {"inner": rng.choice(["4x4x4x4", "2x4x4x4", "4x4x4x2"])} if op == "nested" else {}
    return _case(None, op, text(n), text(blk), nrhs, prec, kappa1=round(rng.uniform(0.1180, 0.1200), 4),
                 kappa2=round(rng.uniform(0.1201, 0.1210), 4), **more)


def _ints(text):
    return tuple(int(v) for v in text.split("x"))


# ------------------------------------------------------------------ inputs
def _mul3(a, b):
    return (a.unsqueeze(-1) * b.unsqueeze(-3)).sum(-2)


def _links(V, gen):
    """SU(3) links exp(i EPS H), H = sum_a h_a lambda_a / 2 with h_a ~ N(0, 1), canonical [4, V, 3, 3]."""
    h = torch.randn((4, V, 8), generator=gen, device="cuda", dtype=torch.float64) / 2
    H = torch.zeros((4, V, 3, 3), device="cuda", dtype=torch.complex128)
    for k, (i, j) in enumerate([(0, 1), (0, 2), (1, 2)]):
        z = torch.complex(h[..., 2 * k], -h[..., 2 * k + 1])
        H[..., i, j], H[..., j, i] = z, z.conj()
    H[..., 0, 0] = h[..., 6] + h[..., 7] / math.sqrt(3)
    H[..., 1, 1] = -h[..., 6] + h[..., 7] / math.sqrt(3)
    H[..., 2, 2] = -2 * h[..., 7] / math.sqrt(3)
    X = H.mul_(1j * EPS / 4)
    U = torch.eye(3, device="cuda", dtype=torch.complex128).expand_as(X)
    one = U
    for k in range(12, 0, -1):  # Horner form of the exponential series
        U = one + _mul3(X, U) / k
    return _mul3(_mul3(U, U), _mul3(U, U))


def _inputs(case, seed):
    """Links and noise (or spinors) of one configuration, from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    V = math.prod(_ints(case["lat"]))
    U = _links(V, gen)
    shape = (case["nrhs"], V, 4, 3)
    if case["op"] in ("estimate", "gradient", "nested"):
        shape = (1,) + shape  # one interpolation step
    return U, torch.randn(shape, generator=gen, device="cuda", dtype=torch.complex128)


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case = case
    U, s.v = _inputs(case, seed)
    s.ctx = dd.Context(U, _ints(case["lat"]), _ints(case["blk"]), -1, CSW)
    if case["op"] == "nested":
        s.inner = dd.Context(U, _ints(case["lat"]), _ints(case["inner"]), -1, CSW)
    if case["op"] == "gradient":
        s.links = U.requires_grad_()
        s.kappa2 = torch.tensor(case["kappa2"], dtype=torch.float64, requires_grad=True)
    return s


def run(s):
    c, prec = s.case, PREC[s.case["prec"]]
    if c["op"] == "dslash":
        return s.ctx.dslash_apply(c["kappa2"], s.v, prec=prec)
    if c["op"] == "block_solve":
        return s.ctx.block_solve(dd.BLACK, c["kappa2"], s.v, tol=c["tol"], prec=prec)[0]
    if c["op"] == "solve":
        return s.ctx.solve(c["kappa2"], s.v, tol=c["tol"], prec=prec)[0]
    if c["op"] == "gradient":
        x = autograd.exponents(s.ctx, c["kappa1"], s.kappa2, s.links, s.v, tol=c["tol"], prec=prec)
        lw = autograd.log_w_gl(x)
        dk, dU = torch.autograd.grad(lw, [s.kappa2, s.links])
        return {"x": x.detach(), "log_w": lw.detach(), "dkappa2": dk, "dU": dU}
    if c["op"] == "nested":
        r = s.ctx.det_ratio_nested(s.inner, dd.BLACK, c["kappa1"], c["kappa2"], s.v, tol=c["tol"], prec=prec)
        return {"x": r["x"], "log_w": r["log_w"]}
    r = s.ctx.det_ratio_estimate(c["kappa1"], c["kappa2"], s.v, op=dd.OP_SCHUR, tol=c["tol"], prec=prec)
    return {"x": r["x"], "log_w": r["log_w_gl"]}


def work(case):
    """Bytes: right-hand sides and results at the FP64 boundary, links and clover in the working
    precision.  Flops: 1980 per site and operator application (eight hops at 180, clover 540); the
    Krylov solves take about 8 applications per decade globally and 5 in a block at these masses."""
    V, n = math.prod(_ints(case["lat"])), case["nrhs"]
    field = 192.0 * V * n
    coef = V * 144.0 * (8 if case["prec"] == "fp64" else 4)
    decades = -math.log10(case["tol"])
    glob, block = 8 * decades, 0.5 * 5 * decades  # (block solves work on half the sites)
    apps = {"dslash": 1, "block_solve": block, "solve": glob, "estimate": glob + 4 * block, "nested": 5 * block / 2,
            "gradient": 3 * glob + 14 * block}[case["op"]]
    out = {"dslash": field, "block_solve": field, "solve": field, "estimate": 8.0 * n, "nested": 8.0 * n,
           "gradient": 8.0 * n + 576.0 * V}[case["op"]]
    return {"bytes": field + out + coef, "flops": 1980.0 * V * n * apps}


def tolerance(case):
    """About four times what the results are off from exact()."""
    if case["op"] == "dslash":
        # sums of about 50 products per component in another order: 2e-16 and 1.1e-7
        return {"rel": 1e-15} if case["prec"] == "fp64" else {"rel": 5e-7}
    # solves stop at the relative residual tol, wherever their iterates happen to stand: solutions are
    # 0.5 to 3.5 tol off, exponents (sums over the lattice) 0.05 tol, and the weights exp(-x) of the
    # gradient carry the absolute error of x: 30 tol
    return {"rel": {"estimate": 0.5, "nested": 0.5, "gradient": 120.0}.get(case["op"], 15.0) * case["tol"]}


# ------------------------------------------------------------------ the same in plain 64-bit torch
# Fields are [4 spin, 3 colour, nrhs, T, L1, L2, L3], links [4, 3, 3, T, L1, L2, L3].  Chiral basis:
# g0 = [[0, -1], [-1, 0]], gk = [[0, -i s_k], [i s_k, 0]].
_UP = [((2, -1), (3, -1)), ((3, -1j), (2, -1j)), ((3, -1), (2, 1)), ((2, -1j), (3, 1j))]    # (g psi)_0, (g psi)_1
_DOWN = [((0, -1), (1, -1)), ((1, 1j), (0, 1j)), ((1, 1), (0, -1)), ((0, 1j), (1, -1j))]    # (g psi)_2, (g psi)_3


def _shift(f, mu, step, bc=1):
    """f(x + step mu); the part that crosses the time boundary times bc."""
    f = torch.roll(f, -step, dims=f.dim() - 4 + mu)
    if mu == 0 and bc != 1:
        sign = torch.ones(f.shape[-4], dtype=torch.float64, device=f.device)
        sign[-1 if step > 0 else 0] = bc
        f = f * sign.view(-1, 1, 1, 1)
    return f


def _mat(a, b):
    return [[sum(a[i][k] * b[k][j] for k in range(3)) for j in range(3)] for i in range(3)]


def _dag(a):
    return [[a[j][i].conj() for j in range(3)] for i in range(3)]


class _Operator:
    """D(m) = (4 + m) + C - H/2 of links U (canonical [4, V, 3, 3]), block structure lat / blk."""

    def __init__(self, U, lat, blk):
        self.lat, self.blk, self.device = lat, blk, U.device
        u = U.permute(0, 2, 3, 1).reshape(4, 3, 3, *lat)
        self.U = [[[u[m, i, j] for j in range(3)] for i in range(3)] for m in range(4)]
        self.C = self._clover()
        co = [torch.arange(n, device=U.device).view([-1 if k == m else 1 for k in range(4)]) for m, n in enumerate(lat)]
        n = [(c // b) for c, b in zip(co, blk)]
        self.colour = (n[0] + n[1] + n[2] + n[3]) % 2
        face = torch.zeros(lat, dtype=torch.bool, device=U.device)
        self.stay = []  # whether the hop x -> x + mu stays inside the block of x
        for c, b in zip(co, blk):
            face = face | (c % b == 0) | (c % b == b - 1)
            self.stay.append((c % b != b - 1).double())
        self.P = (face & (self.colour == 0)).double()

    def _clover(self):
        """The two Hermitian 6x6 chiral blocks, [block][row][column], rows 3 spin + colour."""
        def sh(m, *moves):
            f = self.U[m]
            for mu, step in moves:
                f = [[_shift(f[i][j], mu, step) for j in range(3)] for i in range(3)]
            return f

        F = {}
        for m in range(4):
            for n in range(m + 1, 4):
                q = [_mat(_mat(sh(m), sh(n, (m, 1))), _mat(_dag(sh(m, (n, 1))), _dag(sh(n)))),
                     _mat(_mat(sh(n), _dag(sh(m, (m, -1), (n, 1)))), _mat(_dag(sh(n, (m, -1))), sh(m, (m, -1)))),
                     _mat(_mat(_dag(sh(m, (m, -1))), _dag(sh(n, (m, -1), (n, -1)))), _mat(sh(m, (m, -1), (n, -1)), sh(n, (n, -1)))),
                     _mat(_mat(_dag(sh(n, (n, -1))), sh(m, (n, -1))), _mat(sh(n, (m, 1), (n, -1)), _dag(sh(m))))]
                s = [[q[0][i][j] + q[1][i][j] + q[2][i][j] + q[3][i][j] for j in range(3)] for i in range(3)]
                F[m, n] = [[(s[i][j] - s[j][i].conj()) / 8 for j in range(3)] for i in range(3)]
        # sigma_0k = diag(s_k, -s_k), sigma_jk = -eps_jkl diag(s_l, s_l)
        C = []
        for sg in (1, -1):
            E = [[[sg * F[0, 1][i][j] - F[2, 3][i][j] for j in range(3)] for i in range(3)],
                 [[sg * F[0, 2][i][j] + F[1, 3][i][j] for j in range(3)] for i in range(3)],
                 [[sg * F[0, 3][i][j] - F[1, 2][i][j] for j in range(3)] for i in range(3)]]
            h = 0.5j * CSW
            C.append([[h * (E[2][i % 3][j % 3] * (1 if i < 3 else -1) if i // 3 == j // 3 else
                            E[0][i % 3][j % 3] + (-1j if i < 3 else 1j) * E[1][i % 3][j % 3]) for j in range(6)]
                      for i in range(6)])
        return C

    def hop(self, psi, keep):
        """H psi; keep: "all", "stay" (inside the blocks) or "cross" (through their faces)."""
        out = [[0] * 3 for _ in range(4)]
        for mu in range(4):
            w = 1.0 if keep == "all" else self.stay[mu] if keep == "stay" else 1.0 - self.stay[mu]
            for step, sg in ((1, -1), (-1, 1)):  # (1 - g) U psi(x + mu), (1 + g) U^+(x - mu) psi(x - mu)
                src = _shift(psi, mu, 1, -1) if step > 0 else psi
                h = [src[s] + (sg * _UP[mu][s][1]) * src[_UP[mu][s][0]] for s in (0, 1)]
                u = self.U[mu] if step > 0 else _dag(self.U[mu])
                k = torch.stack([torch.stack([w * (u[a][0] * h[s][0] + u[a][1] * h[s][1] + u[a][2] * h[s][2])
                                              for a in range(3)]) for s in (0, 1)])
                if step < 0:
                    k = _shift(k, mu, -1, -1)
                for s in (0, 1):
                    p, z = _DOWN[mu][s]
                    for a in range(3):
                        out[s][a] = out[s][a] + k[s, a]
                        out[2 + s][a] = out[2 + s][a] + (sg * z) * k[p, a]
        return torch.stack([torch.stack(o) for o in out])

    def diag(self, psi, mass):
        f = psi.reshape(2, 6, *psi.shape[2:])
        out = [[(4 + mass) * f[b, i] + sum(self.C[b][i][j] * f[b, j] for j in range(6)) for i in range(6)] for b in (0, 1)]
        return torch.stack([torch.stack(o) for o in out]).reshape(psi.shape)

    def only(self, psi, colour):
        return psi * (self.colour == colour).double()

    def D(self, psi, mass, colour=None):
        """D psi, or the Dirichlet block operator of one colour on that colour's sites."""
        return self.diag(psi, mass) - 0.5 * self.hop(psi, "all" if colour is None else "stay")

    def cross(self, psi, to):
        """D_wb (to = 1) or D_bw (to = 0): hops through block faces into one colour."""
        return self.only(-0.5 * self.hop(psi, "cross"), to)

    def field(self, v):
        return v.reshape(-1, *self.lat, 4, 3).permute(5, 6, 0, 1, 2, 3, 4).contiguous()

    def canonical(self, f, shape):
        return f.permute(2, 3, 4, 5, 6, 0, 1).reshape(shape)


def _dot(a, b):
    return (a.conj() * b).sum(dim=(0, 1, 3, 4, 5, 6))


def _bicgstab(A, b, tol=3e-15):
    """x with ||b - A x|| <= tol ||b|| for each right-hand side, restarted on the true residual."""
    v = lambda z: z.view(-1, 1, 1, 1, 1)  # noqa: E731
    safe = lambda z: torch.where(z.abs() > 0, z, torch.ones_like(z))  # noqa: E731
    x, r, bb = torch.zeros_like(b), b.clone(), _dot(b, b).real
    for _ in range(4):
        goal = tol ** 2 * bb
        rh, p, e, rho = r.clone(), r.clone(), torch.zeros_like(b), _dot(r, r)
        stop = torch.maximum(goal, 1e-20 * rho.real)
        for k in range(500):
            y = A(p)
            al = rho / safe(_dot(rh, y))
            s = r - v(al) * y
            t = A(s)
            om = _dot(t, s) / safe(_dot(t, t))
            e += v(al) * p + v(om) * s
            r = s - v(om) * t
            if k % 4 == 3 and bool((_dot(r, r).real <= stop).all()):
                break
            new = _dot(rh, r)
            p = r + v(new / safe(rho) * al / safe(om)) * (p - v(om) * y)
            rho = new
        x += e
        r = b - A(x)
        if bool((_dot(r, r).real <= goal).all()):
            break
    return x


class _Inverse(torch.autograd.Function):
    """D(m)^-1 b (or the block inverse of one colour), differentiable in b, the links and the mass."""

    @staticmethod
    def forward(ctx, U, b, lat, blk, mass, colour):
        O = _Operator(U, lat, blk)
        x = _bicgstab(lambda f: O.D(f, float(mass), colour), b if colour is None else O.only(b, colour))
        ctx.save_for_backward(U, x)
        ctx.more = (lat, blk, float(mass), colour)
        return x

    @staticmethod
    def backward(ctx, gx):
        U, x = ctx.saved_tensors
        lat, blk, mass, colour = ctx.more
        O = _Operator(U, lat, blk)
        g5 = torch.tensor([1.0, 1, -1, -1], dtype=torch.float64, device=U.device).view(4, 1, 1, 1, 1, 1, 1)
        rhs = g5 * gx  # D^+ = g5 D g5
        z = g5 * _bicgstab(lambda f: O.D(f, mass, colour), rhs if colour is None else O.only(rhs, colour))
        with torch.enable_grad():
            W = U.detach().requires_grad_()
            y = _Operator(W, lat, blk).D(x, mass, colour)
            gU, = torch.autograd.grad(-(z.conj() * y).real.sum(), W)
        return gU, z, None, None, -(z.conj() * x).real.sum() if ctx.needs_input_grad[4] else None, None


def _mass(kappa):
    return 1.0 / (2.0 * kappa) - 4.0


def _exponents(U, case, v, m1, m2):
    """Schur exponents 2 Re<e, y> + ||y||^2 of y = (Dhat(m2)^-1 Dhat(m1) - 1) e."""
    lat, blk = _ints(case["lat"]), _ints(case["blk"])
    O = _Operator(U, lat, blk)
    inv = lambda b, m, c=None: _Inverse.apply(U, b, lat, blk, m, c)  # noqa: E731
    e = O.field(v) * O.P
    w = inv(O.cross(e, 1), m1, 1)
    g = inv(O.cross(inv(w, m2, 1), 0) + inv(O.cross(w, 0), m1, 0), m2, 0) * ((m1 - m2) * O.P)
    y = g - O.P * inv(O.cross(g, 1), m2)
    return 2 * _dot(e, y).real + _dot(y, y).real


def _exponents_nested(U, case, v, m1, m2):
    """The same for the black outer blocks split by the inner ones: hops cut to those blocks."""
    lat = _ints(case["lat"])
    O, I = _Operator(U, lat, _ints(case["blk"])), _Operator(U, lat, _ints(case["inner"]))
    here = (O.colour == 0).double()
    inv = lambda b, m, c: _bicgstab(lambda f: I.D(f, m, c), I.only(b, c))  # noqa: E731
    P = I.P * here
    cut = lambda f, to: here * I.cross(here * f, to)  # noqa: E731
    # (a hop through an inner face between two black outer blocks does not exist: they never touch)
    e = I.field(v) * P
    w = inv(cut(e, 1), m1, 1)
    g = inv(cut(inv(w, m2, 1), 0) + inv(cut(w, 0), m1, 0), m2, 0) * ((m1 - m2) * P)
    y = g - P * _bicgstab(lambda f: O.D(f, m2, 0), cut(g, 1))
    return 2 * _dot(e, y).real + _dot(y, y).real


def exact(case, seed):
    op, pairs = case["op"], math.prod(_ints(case["lat"])) * case["nrhs"]
    if pairs > {"dslash": 2e7, "block_solve": 1e7, "solve": 1e7, "estimate": 3e6, "gradient": 1.2e6, "nested": 1.2e6}[op]:
        return None  # (over about 20 seconds)
    U, v = _inputs(case, seed)
    m1, m2 = _mass(case["kappa1"]), _mass(case["kappa2"])
    if op == "gradient":
        U.requires_grad_()
        k2 = torch.tensor(case["kappa2"], dtype=torch.float64, device="cuda", requires_grad=True)
        x = _exponents(U, case, v, m1, _mass(k2))
        lw = torch.logsumexp(-x, 0) - math.log(x.numel())
        dk, dU = torch.autograd.grad(lw, [k2, U])
        return {"x": x.detach().view(1, -1), "log_w": lw.detach(), "dkappa2": dk, "dU": dU}
    with torch.no_grad():
        if op in ("estimate", "nested"):
            x = (_exponents if op == "estimate" else _exponents_nested)(U, case, v, m1, m2).cpu().numpy()
            top = float(np.max(-x))
            return {"x": x[None], "log_w": top + math.log(float(np.mean(np.exp(-x - top))))}
        O = _Operator(U, _ints(case["lat"]), _ints(case["blk"]))
        f = O.field(v)
        if op == "dslash":
            f = O.D(f, m2)
        elif op == "solve":
            f = _bicgstab(lambda z: O.D(z, m2), f)
        else:
            f = _bicgstab(lambda z: O.D(z, m2, 0), O.only(f, 0))
        return O.canonical(f, v.shape)
