"""Performance cases: the work a program does with this framework, through its public entry points.

A case is a dict of plain values; ``listed()`` gives the standing cases, ``draw(rng)`` further ones of
the same ranges.  ``prepare`` makes what a program has before the call (perturbed unit-cube mesh,
operator, input vectors on the GPU), ``run`` is one pass, ``work`` the bytes and operations one pass
cannot do without, and ``exact`` the same result in plain torch, 64-bit, by dense 1D contractions.

Paths (field ``path``):
  apply    y = A x of the hexahedral operator: BP1 (mass), BP3 (diffusion, Gauss), BP5 / BP6 (diffusion,
           collocated; BP6 with three components), one or several right-hand sides, float64 or float32,
           optionally with in-kernel factors ("otf") or the deterministic scatter ("det")
  adjoint  variable-coefficient diffusion with its gradients in u and kappa (one training step's work)
  cg       a fixed number of FP64 CG iterations
  mg       one p-multigrid V-cycle
  tet      y = A x of the tetrahedral P_p operator
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2109_05072_amd as mf

_BASE = {"path": "apply", "kind": "diffusion", "quad": "gauss", "p": 3, "nex": 6, "ney": 6, "nez": 6, "ncomp": 1,
         "nrhs": 1, "dtype": "float64", "dirichlet": True, "option": "", "iters": 0}


def _case(name=None, **kw):
    c = dict(_BASE, **kw)
    return c if name is None else dict(c, name=name)


def _cube(p, nodes):
    """Elements per direction of a cubic mesh with about `nodes` nodes."""
    return max(1, int(round((nodes ** (1.0 / 3.0) - 1.0) / p)))


def listed():
    def cube(p, nodes):
        ne = _cube(p, nodes)
        return dict(p=p, nex=ne, ney=ne, nez=ne)

    return [
        # the smallest problems (a coarse level, a unit test, a strongly scaled rank): launch latency
        _case("bp3_small_p3", p=3, nex=6, ney=6, nez=6),
        # the headline sweep's size, low, and high order: one apply at about 1e7 nodes
        _case("bp3_p3", **cube(3, 1e7)),
        _case("bp3_p7", **cube(7, 1e7)),
        # an ordinary problem on a ragged box (odd element counts in every direction), about 2e6 nodes
        _case("bp3_p5_ragged", p=5, nex=37, ney=19, nez=23),
        # the operator inside mixed-precision solvers, about 1e7 nodes
        _case("bp3_p4_f32", dtype="float32", **cube(4, 1e7)),
        # BP1: the mass operator (projections, explicit time steps), about 1e7 nodes
        _case("bp1_p4", kind="mass", dirichlet=False, **cube(4, 1e7)),
        # BP5 with eight right-hand sides (block solvers, ensembles), about 1e7 nodes
        _case("bp5_p6_8rhs", quad="gll", nrhs=8, **cube(6, 1e7)),
        # BP6 (three components) with a few right-hand sides on a ragged box, about 1e6 nodes
        _case("bp6_p3_4rhs_ragged", quad="gll", ncomp=3, nrhs=4, p=3, nex=41, ney=27, nez=33),
        # the forward and backward pass of a coefficient inversion, about 1e7 nodes
        _case("adjoint_p4", path="adjoint", **cube(4, 1e7)),
        # the solver half of the headline metric: CG iterations at about 1e6 nodes
        _case("cg_p5", path="cg", iters=30, **cube(5, 1e6)),
        # one preconditioner application of the multigrid solver, about 1.4e6 nodes, levels 7, 3, 1
        _case("mg_p7", path="mg", p=7, nex=16, ney=16, nez=16),
        # the tetrahedral operator, about 1e7 nodes
        _case("tet_p3", path="tet", **cube(3, 1e7)),
    ]


def _box(rng, p, nodes):
    """Element counts of a box with about `nodes` nodes whose sides differ."""
    ne = (nodes ** (1.0 / 3.0) - 1.0) / p
    ax = [max(1, int(round(ne * rng.uniform(0.75, 1.2)))) for _ in range(3)]
    return dict(nex=ax[0], ney=ax[1], nez=ax[2])


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    f = rng.random()
    if f < 0.40:  # one vector, any operator
        p = rng.randint(1, 8)
        c = dict(p=p, kind="diffusion" if rng.random() < 0.7 else "mass", quad="gauss" if rng.random() < 0.75 else "gll",
                 dtype="float64" if rng.random() < 0.75 else "float32", dirichlet=rng.random() < 0.75,
                 **_box(rng, p, _log(rng, 2e3, 8e6)))
        o = rng.random()
        if o < 0.10:
            c["option"] = "det"
        elif o < 0.25 and c["kind"] == "diffusion" and c["dtype"] == "float64":
            c["option"] = "otf"
        return _case(**c)
    if f < 0.60:  # several vectors, collocated
        p = rng.randint(2, 8)
        nc, nr = rng.choice([1, 3]), rng.randint(2, 16)
        return _case(p=p, quad="gll", ncomp=nc, nrhs=nr, dtype="float64" if rng.random() < 0.8 else "float32",
                     **_box(rng, p, min(6e6, _log(rng, 1e5, 6e7) / (nc * nr))))
    if f < 0.70:
        p = rng.randint(2, 6)
        return _case(path="adjoint", p=p, **_box(rng, p, _log(rng, 3e4, 6e6)))
    if f < 0.78:
        p = rng.randint(2, 8)
        return _case(path="cg", p=p, iters=rng.randint(10, 30), **_box(rng, p, _log(rng, 2e4, 8e5)))
    if f < 0.84:
        p = rng.randint(2, 8)
        return _case(path="mg", p=p, **_box(rng, p, _log(rng, 3e4, 1e6)))
    p = rng.randint(1, 6)
    return _case(path="tet", p=p, dirichlet=rng.random() < 0.75, **_box(rng, p, _log(rng, 1e4, 8e6)))


# --- a program's side ---------------------------------------------------------------------------------


def _vertices(c, seed):
    """Host [(nex+1)(ney+1)(nez+1), 3] float64: a uniform grid of the unit cube, interior vertices shifted by +-0.1 h."""
    ne = (c["nex"], c["ney"], c["nez"])
    rng = np.random.default_rng([seed, 1])
    v = np.empty((ne[2] + 1, ne[1] + 1, ne[0] + 1, 3))
    v[..., 0] = np.linspace(0.0, 1.0, ne[0] + 1)
    v[..., 1] = np.linspace(0.0, 1.0, ne[1] + 1)[:, None]
    v[..., 2] = np.linspace(0.0, 1.0, ne[2] + 1)[:, None, None]
    inner = v[1:-1, 1:-1, 1:-1]
    inner += (rng.random(inner.shape) - 0.5) * (0.2 / np.array(ne, dtype=float))
    return np.ascontiguousarray(v.reshape(-1, 3))


def _q(c):
    return c["p"] + 2 if c["quad"] == "gauss" else c["p"] + 1


def _nodes(c, p=None):
    p = c["p"] if p is None else p
    return (p * c["nex"] + 1) * (p * c["ney"] + 1) * (p * c["nez"] + 1)


def _elems(c):
    return c["nex"] * c["ney"] * c["nez"]


def _inputs(c, seed):
    """Device inputs: x (apply, cg, mg, tet), and for the adjoint u, kappa, f; uniform in [-1, 1], kappa log-uniform."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2 + 1)

    def uni(*shape):
        return torch.rand(*shape, dtype=torch.float64, device="cuda", generator=g) * 2.0 - 1.0

    n = _nodes(c)
    if c["path"] == "adjoint":
        return {"u": uni(n), "kappa": torch.exp(0.5 * uni(_elems(c), _q(c) ** 3)), "f": uni(n)}
    if c["path"] in ("cg", "mg"):  # a right-hand side of the masked operator: zero on the boundary
        b = torch.zeros(c["p"] * c["nez"] + 1, c["p"] * c["ney"] + 1, c["p"] * c["nex"] + 1, dtype=torch.float64, device="cuda")
        inner = b[1:-1, 1:-1, 1:-1]
        inner.copy_(uni(*inner.shape))
        return {"x": b.reshape(-1)}
    nvec = c["nrhs"] * c["ncomp"]
    x = uni(n) if nvec == 1 else uni(n, c["nrhs"], c["ncomp"])
    return {"x": x.to(getattr(torch, c["dtype"]))}


def prepare(case, seed):
    c = case
    vert = _vertices(c, seed)
    s = {"case": c, **_inputs(c, seed)}
    if c["path"] == "tet":
        s["op"] = mf.TetOperator(c["nex"], c["ney"], c["nez"], c["p"], vert, dirichlet=c["dirichlet"])
    else:
        s["op"] = mf.Operator(c["nex"], c["ney"], c["nez"], c["p"], vert, kind=c["kind"], quad=c["quad"], ncomp=c["ncomp"],
                              dirichlet=c["dirichlet"], variable_kappa=c["path"] == "adjoint",
                              f32=c["dtype"] == "float32", otf=c["option"] == "otf",
                              deterministic=c["option"] == "det")
    if c["path"] == "adjoint":
        s["u"].requires_grad_(True)
        s["kappa"].requires_grad_(True)
    elif c["path"] == "mg":
        s["op"].mg_setup()
    if c["path"] in ("apply", "mg", "tet"):
        s["y"] = torch.empty_like(s["x"])
    return s


def run(state):
    s, c = state, state["case"]
    op = s["op"]
    if c["path"] in ("apply", "tet"):
        return op.apply(s["x"], s["y"])
    if c["path"] == "mg":
        return op.mg_apply(s["x"], s["y"])
    if c["path"] == "cg":
        return op.cg(s["x"], maxit=c["iters"], exact_iters=True, rtol=0.0).x
    y = mf.diffusion(s["u"], s["kappa"], op)
    loss = 0.5 * ((y - s["f"]) ** 2).sum()
    gu, gk = torch.autograd.grad(loss, [s["u"], s["kappa"]])
    return y.detach(), gu, gk


# --- what a pass cannot do without --------------------------------------------------------------------


def _apply_work(c, p, q, nvec, s):
    """One apply: x in, y out, the operator's stored factors (none with "otf"); sum-factorized operations."""
    E, P = _elems(c), p + 1
    g = 6 if c["kind"] == "diffusion" else 1
    stored = 0 if c["option"] == "otf" else s * g * E * q ** 3
    interp = 0 if q == P else 4 * (q * P ** 3 + q * q * P * P + q ** 3 * P)
    flops = interp + (12 * q ** 4 + 15 * q ** 3 if g == 6 else q ** 3)
    return 2 * s * _nodes(c, p) * nvec + stored, E * flops * nvec


def work(case):
    c = case
    p, q, N, E = c["p"], _q(c), _nodes(c), _elems(c)
    s = 4 if c["dtype"] == "float32" else 8
    if c["path"] == "apply":
        b, f = _apply_work(c, p, q, c["nrhs"] * c["ncomp"], s)
    elif c["path"] == "adjoint":
        b1, f1 = _apply_work(c, p, q, 1, 8)
        pts = 8 * E * q ** 3
        # forward and the u-gradient: an apply and kappa each; the kappa-gradient: factors, u and r in, kappa-sized out
        b = 2 * (b1 + pts) + (b1 + pts)
        f = 3 * f1
    elif c["path"] == "cg":
        b1, f1 = _apply_work(c, p, q, 1, 8)
        # per iteration the apply, x, r, p, Ap in and x, r out, then r, p in and p out
        b, f = c["iters"] * (b1 + 72 * N), c["iters"] * (f1 + 12 * N)
    elif c["path"] == "mg":
        b = f = 0
        while True:
            applies = 6 if p > 1 else 7
            b1, f1 = _apply_work(c, p, p + 2 if c["quad"] == "gauss" else p + 1, 1, 8)
            # per smoothing step x, d, r, Ad, dinv in and x, d, r out
            b += applies * b1 + 64 * applies * _nodes(c, p)
            f += applies * f1
            if p == 1:
                break
            p //= 2
    else:
        # vertices, x, y; the gradient of a P_p field lies in P_{p-1}: 3 products with dim(P_{p-1}) rows each way
        P, M = (p + 1) * (p + 2) * (p + 3) // 6, p * (p + 1) * (p + 2) // 6
        b = 16 * N + 24 * (c["nex"] + 1) * (c["ney"] + 1) * (c["nez"] + 1)
        f = 6 * E * (12 * M * P + 15 * M)
    return {"bytes": b, "flops": f}


# --- the same results in plain torch, 64-bit ----------------------------------------------------------


def _lobatto(n):
    """n Gauss-Lobatto points and weights."""
    leg = np.polynomial.legendre.Legendre.basis(n - 1)
    d, dd = leg.deriv(), leg.deriv(2)
    x = np.sort(d.roots().real) if n > 2 else np.zeros(0)
    for _ in range(4):
        x = x - d(x) / dd(x) if n > 2 else x
    x = np.concatenate([[-1.0], x, [1.0]])
    return x, 2.0 / (n * (n - 1) * leg(x) ** 2)


def _lagrange(xn, xe):
    """Values [e][n] and derivatives [e][n] of the Lagrange polynomials on xn at the points xe."""
    n = len(xn)
    B, D = np.ones((len(xe), n)), np.zeros((len(xe), n))
    for i in range(n):
        den = np.prod([xn[i] - xn[m] for m in range(n) if m != i])
        for e, x in enumerate(xe):
            B[e, i] = np.prod([x - xn[m] for m in range(n) if m != i]) / den
            D[e, i] = sum(np.prod([x - xn[k] for k in range(n) if k not in (i, m)]) for m in range(n) if m != i) / den
    return B, D


def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(_dev())


def _ax(M, U, axis):
    """Contract axis `axis` (negative) of U with the rows of M."""
    return torch.tensordot(U, M, dims=([U.dim() + axis], [1])).movedim(-1, axis)


class _Plain:
    """One order's operator on a structured mesh: element fields are [ez, ey, ex, v, z, y, x]."""

    def __init__(self, c, vert, p, quad):
        self.c, self.p, self.P = c, p, p + 1
        self.ne = (c["nez"], c["ney"], c["nex"])
        xn, wn = _lobatto(p + 1)
        xq, wq = np.polynomial.legendre.leggauss(p + 2) if quad == "gauss" else (xn, wn)
        B, D = _lagrange(xn, xq)
        self.B, self.D, self.xn = _t(B), _t(D), xn
        self.Q = len(xq)
        L = _t(np.stack([(1 - xq) / 2, (1 + xq) / 2], 1))
        dL = _t(np.tile([-0.5, 0.5], (self.Q, 1)))
        V = _t(vert).reshape(self.ne[0] + 1, self.ne[1] + 1, self.ne[2] + 1, 3)
        self.C = V.unfold(0, 2, 1).unfold(1, 2, 1).unfold(2, 2, 1)  # [ez, ey, ex, 3, z, y, x]
        self.L, self.dL = L, dL
        w = _t(wq)
        self.w = w[:, None, None] * w[None, :, None] * w[None, None, :]
        n = [p * m + 1 for m in self.ne]
        self.n = n
        m = torch.ones(n, dtype=torch.float64, device=_dev())
        if c["dirichlet"]:
            m[0], m[-1], m[:, 0], m[:, -1], m[:, :, 0], m[:, :, -1] = 0, 0, 0, 0, 0, 0
        self.mask = m

    def factors(self, z):
        """Mass weight or the six factors (3x3, symmetric) at the points of element layer z."""
        C, L, dL = self.C[z:z + 1], self.L, self.dL
        J = [_ax(a, _ax(b, _ax(k, C, -3), -2), -1) for k, b, a in ((L, L, dL), (L, dL, L), (dL, L, L))]
        J = [j.movedim(3, -1) for j in J]  # columns dx/dr, dx/ds, dx/dt: [.., z, y, x, 3]
        rows = [torch.linalg.cross(J[1], J[2]), torch.linalg.cross(J[2], J[0]), torch.linalg.cross(J[0], J[1])]
        det = (J[0] * rows[0]).sum(-1)
        if self.c["kind"] == "mass":
            return self.w * det
        s = self.w / det
        return [[s * (rows[a] * rows[b]).sum(-1) for b in range(3)] for a in range(3)]

    def gather(self, x, z):
        """Element values of layer z; x: [Z, Y, X, v]."""
        p, P = self.p, self.P
        u = x[z * p:z * p + P].unfold(0, P, p).unfold(1, P, p).unfold(2, P, p)
        return u

    def scatter(self, y, e, z):
        """y[Z, Y, X, v] += element values of layer z, overlapping faces summed."""
        p = self.p
        out = e[0]  # [ey, ex, v, k, j, i]
        ey, ex, v = out.shape[:3]
        a = torch.zeros(ey, v, self.P, self.P, self.n[2], dtype=e.dtype, device=e.device)
        o = out.permute(0, 2, 3, 4, 1, 5)  # [ey, v, k, j, ex, i]
        a[..., :-1] += o[..., :p].reshape(*a.shape[:-1], -1)
        a[..., p::p] += o[..., p]
        b = torch.zeros(v, self.P, self.n[1], self.n[2], dtype=e.dtype, device=e.device)
        o = a.permute(1, 2, 0, 3, 4)  # [v, k, ey, j, X]
        b[:, :, :-1] += o[:, :, :, :p].reshape(v, self.P, -1, self.n[2])
        b[:, :, p::p] += o[:, :, :, p]
        y[z * p:z * p + self.P] += b.permute(1, 2, 3, 0)

    def grad(self, u):
        B, D = self.B, self.D
        ux = _ax(B, _ax(B, u, -3), -2)
        return [_ax(D, ux, -1), _ax(B, _ax(D, _ax(B, u, -3), -2), -1), _ax(B, _ax(B, _ax(D, u, -3), -2), -1)]

    def grad_t(self, v):
        B, D = self.B.T, self.D.T
        return (_ax(B, _ax(B, _ax(D, v[0], -1), -2), -3) + _ax(B, _ax(D, _ax(B, v[1], -1), -2), -3)
                + _ax(D, _ax(B, _ax(B, v[2], -1), -2), -3))

    def apply(self, x, kappa=None):
        """x: [N] or [N, v] float64."""
        v = x.reshape(*self.n, -1) * self.mask[..., None]
        y = torch.zeros_like(v)
        for z in range(self.ne[0]):
            u, G = self.gather(v, z), self.factors(z)
            if self.c["kind"] == "mass":
                B, Bt = self.B, self.B.T
                f = _ax(B, _ax(B, _ax(B, u, -3), -2), -1) * G[:, :, :, None]
                e = _ax(Bt, _ax(Bt, _ax(Bt, f, -1), -2), -3)
            else:
                g = self.grad(u)
                k = 1.0 if kappa is None else self.points(kappa, z)[:, :, :, None]
                e = self.grad_t([k * sum(G[a][b][:, :, :, None] * g[b] for b in range(3)) for a in range(3)])
            self.scatter(y, e, z)
        return (y * self.mask[..., None]).reshape(x.shape)

    def points(self, k, z):
        """Per-point values [E, Q^3] of element layer z as [1, ey, ex, z, y, x]."""
        return k.reshape(*self.ne, self.Q, self.Q, self.Q)[z:z + 1]

    def kappa_grad(self, u, r):
        out = []
        uv, rv = (t.reshape(*self.n, 1) * self.mask[..., None] for t in (u, r))
        for z in range(self.ne[0]):
            G = self.factors(z)
            gu, gr = (self.grad(self.gather(t, z)) for t in (uv, rv))
            out.append(sum(G[a][b] * gu[b][:, :, :, 0] * gr[a][:, :, :, 0] for a in range(3) for b in range(3)).reshape(-1))
        return torch.cat(out).reshape(-1, self.Q ** 3)

    def diagonal(self):
        y = torch.zeros(*self.n, 1, dtype=torch.float64, device=_dev())
        B, D = self.B, self.D
        m = ((B * B).T, (B * D).T, (D * D).T)
        for z in range(self.ne[0]):
            G = self.factors(z)
            e = 0.0
            for a in range(3):
                for b in range(3):
                    t = [m[int(a == ax) + int(b == ax)] for ax in range(3)]
                    e = e + _ax(t[2], _ax(t[1], _ax(t[0], G[a][b], -1), -2), -3)
            self.scatter(y, e[:, :, :, None], z)
        return (y[..., 0] * self.mask).reshape(-1)


def _splitmix(n, seed):
    with np.errstate(over="ignore"):
        z = np.uint64((seed * 0x632BE59BD9B4E019) & ((1 << 64) - 1)) + np.arange(n, dtype=np.uint64)
        z = z + np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
    return 2.0 * ((z >> np.uint64(11)).astype(np.float64) / 9007199254740992.0) - 1.0


def _vcycle(c, vert, b):
    """The V-cycle of the entry point's documentation (default options)."""
    orders = [c["p"]]
    while orders[-1] > 1:
        orders.append(max(1, orders[-1] // 2))
    lv = []
    for p in orders:
        A = _Plain(c, vert, p, c["quad"])
        d = A.diagonal()
        dinv = torch.where(d > 0, 1.0 / d, torch.zeros_like(d))
        v = _t(_splitmix(d.numel(), 2024)) * (d > 0)
        v = v / v.norm()
        for _ in range(15):
            av = A.apply(v)
            lam = float((v @ av) / (v @ (d * v)))
            v = dinv * av
            v = v / v.norm()
        lv.append((A, dinv, lam))

    def smooth(l, rhs, x, degree):
        A, dinv, lam = lv[l]
        lo, hi = 0.25 * lam, 1.1 * lam
        theta, delta = 0.5 * (hi + lo), 0.5 * (hi - lo)
        sigma = theta / delta
        r = dinv * (rhs if x is None else rhs - A.apply(x))
        x = torch.zeros_like(rhs) if x is None else x
        d, rho = r / theta, delta / theta
        for k in range(degree):
            x = x + d
            if k + 1 < degree:
                r = r - dinv * A.apply(d)
                new = 1.0 / (2.0 * sigma - rho)
                d, rho = new * rho * d + 2.0 * new / delta * r, new
        return x

    def share(A):
        m = [torch.ones(k, dtype=torch.float64, device=_dev()) for k in A.n]
        for t in m:
            t[A.p:-1:A.p] = 0.5
        return m[0][:, None, None] * m[1][None, :, None] * m[2][None, None, :]

    def move(src, dst, M, x, weighted_out):
        """Element by element through M: prolongation (weights on the output) or restriction (on the input)."""
        v = x.reshape(src.n) * src.mask * (1.0 if weighted_out else share(src))
        y = torch.zeros(*dst.n, 1, dtype=torch.float64, device=_dev())
        for z in range(src.ne[0]):
            dst.scatter(y, _ax(M, _ax(M, _ax(M, src.gather(v[..., None], z), -1), -2), -3), z)
        return (y[..., 0] * dst.mask * (share(dst) if weighted_out else 1.0)).reshape(-1)

    def cycle(l, rhs):
        if l + 1 == len(lv):
            return smooth(l, rhs, None, 8)
        x = smooth(l, rhs, None, 3)
        F, C = lv[l][0], lv[l + 1][0]
        M = _t(_lagrange(C.xn, F.xn)[0])
        xc = cycle(l + 1, move(F, C, M.T.contiguous(), rhs - F.apply(x), False))
        return smooth(l, rhs, x + move(C, F, M, xc, True), 3)

    return cycle(0, b)


def _tet_apply(c, vert, x):
    """Kuhn split: element stiffness = sum over a, b of D_ab int d_a phi_i d_b phi_j, D = |det J| J^-1 J^-T."""
    p, ne = c["p"], (c["nex"], c["ney"], c["nez"])
    lat = [(a, b, d) for d in range(p + 1) for b in range(p + 1 - d) for a in range(p + 1 - d - b)]
    n = np.array(lat)
    # rule: tensor Gauss-Legendre mapped to the tetrahedron, exact beyond the products needed
    t, w = np.polynomial.legendre.leggauss(p + 2)
    t, w = (t + 1) / 2, w / 2
    a, b, d = (m.reshape(-1) for m in np.meshgrid(t, t, t, indexing="ij"))
    W = np.einsum("i,j,k->ijk", w, w, w).reshape(-1) * (1 - b) * (1 - d) ** 2
    X = np.stack([a * (1 - b) * (1 - d), b * (1 - d), d], 1)
    lam = np.concatenate([1 - X.sum(1, keepdims=True), X], 1)
    idx = np.concatenate([p - n.sum(1, keepdims=True), n], 1)

    def R(k, z):
        v, dv = np.ones_like(z), np.zeros_like(z)
        for j in range(k):
            v, dv = v * (z - j) / (j + 1), (dv * (z - j) + v) / (j + 1)
        return v, dv

    G = np.zeros((3, len(W), len(n)))
    for i, m in enumerate(idx):
        f = [R(m[k], p * lam[:, k]) for k in range(4)]
        dl = [p * f[k][1] * np.prod([f[o][0] for o in range(4) if o != k], 0) for k in range(4)]
        for k in range(3):
            G[k, :, i] = dl[k + 1] - dl[0]
    K = _t(np.einsum("aqi,q,bqj->abij", G, W, G))
    V = _t(vert).reshape(ne[2] + 1, ne[1] + 1, ne[0] + 1, 3)
    nn = [p * m + 1 for m in ne]
    mask = torch.ones(nn[2], nn[1], nn[0], dtype=torch.float64, device=_dev())
    if c["dirichlet"]:
        mask[0], mask[-1], mask[:, 0], mask[:, -1], mask[:, :, 0], mask[:, :, -1] = 0, 0, 0, 0, 0, 0
    xm = x.reshape(mask.shape) * mask
    y = torch.zeros_like(xm)
    for pi in ((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)):
        corner = np.zeros((4, 3), dtype=int)
        for k in range(3):
            corner[k + 1:, pi[k]] = 1
        P4 = [V[k[2]:k[2] + ne[2], k[1]:k[1] + ne[1], k[0]:k[0] + ne[0]] for k in corner]
        J = [P4[k] - P4[0] for k in (1, 2, 3)]
        rows = [torch.linalg.cross(J[1], J[2]), torch.linalg.cross(J[2], J[0]), torch.linalg.cross(J[0], J[1])]
        det = (J[0] * rows[0]).sum(-1).abs()
        node = n @ (corner[1:] - corner[0])  # lattice offset of every basis function
        sl = [tuple(slice(int(o[k]), int(o[k]) + p * (ne[k] - 1) + 1, p) for k in (2, 1, 0)) for o in node]
        U = torch.stack([xm[s] for s in sl], -1)
        Y = 0.0
        for i in range(3):
            for j in range(3):
                Y = Y + ((rows[i] * rows[j]).sum(-1) / det)[..., None] * (U @ K[i, j].T)
        for i, s in enumerate(sl):
            y[s] += Y[..., i]
    return (y * mask).reshape(-1)


def exact(case, seed):
    c = case
    vert, s = _vertices(c, seed), {k: v.to(_dev()) for k, v in _inputs(c, seed).items()}
    if c["path"] == "tet":
        return _tet_apply(c, vert, s["x"])
    if c["path"] == "mg":
        return _vcycle(c, vert, s["x"])
    A = _Plain(c, vert, c["p"], c["quad"])
    if c["path"] == "apply":
        x = s["x"].double()
        return A.apply(x.reshape(_nodes(c), -1)).reshape(x.shape)
    if c["path"] == "adjoint":
        y = A.apply(s["u"], s["kappa"])
        r = y - s["f"]
        return y, A.apply(r, s["kappa"]), A.kappa_grad(s["u"], r)
    b = s["x"]
    x, r = torch.zeros_like(b), b.clone()
    d, rr = r.clone(), r @ r
    for _ in range(c["iters"]):
        q = A.apply(d)
        al = rr / (d @ q)
        x, r = x + al * d, r - al * q
        new = r @ r
        d, rr = r + (new / rr) * d, new
    return x
