"""Workloads of the finite-element Hamiltonian filter, as a user's program runs them.

Each case is a dict of plain values.  `prepare` makes its inputs on the GPU
from a seed and the mesh handle and buffers that a program keeps, `run` makes
one pass through the public entry points, `exact` computes the same outputs in
64 bits with dense one-dimensional matrices in torch, without the library.

The operator is H~ = M^-1/2 (K/2 + V) M^-1/2 (+ C D C^T) on a box of cubic
cells of edge 1 bohr with GLL nodes of degree p; "bc" gives a letter per axis
(P periodic, D zero-Dirichlet, N zero-Neumann).  BF16 cell products are left
out: their Ritz values miss the accuracy the filter is used at.
"""
import math

import numpy as np
import torch

import paper_2504_00998_amd as fe
from paper_2504_00998_amd import solver

DEV = "cuda"
F64 = torch.float64
BC = {"D": fe.DIRICHLET, "P": fe.PERIODIC, "N": fe.NEUMANN}
FIELD = 0.005      # Ha/bohr, about the box centre
DEPTH, SIGMA = -3.0, 0.6
R_CUT, R_G = 2.0, 0.5


def _case(name, kind, p, cells, N=1, m=1, bc="PPD", prec="f64", pad=0, sites=0, kx=0.0, ky=0.0):
    c = dict(kind=kind, p=p, nx=cells[0], ny=cells[1], nz=cells[2], bc=bc, N=N, m=m, prec=prec, pad=pad, sites=sites,
             kx=kx, ky=ky)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest problem of the tests: a few hundred launches' worth of latency, hardly any arithmetic
        _case("cube-p3-filter", "filter", 3, (4, 4, 4), N=16, m=20, bc="DDD"),
        # the benchmark's step: potential update and degree-30 filter of the p = 4 slab
        _case("slab-p4-filter", "filter", 4, (24, 24, 48), N=256, m=30),
        # the p = 6 slab of the benchmark, degree 20
        _case("slab-p6-filter", "filter", 6, (16, 16, 32), N=128, m=20),
        # the p = 5 slab with nonlocal projectors in mixed precision, on a box whose blocks fit the card three times
        _case("slab-p5-f32-nonlocal", "filter", 5, (20, 20, 40), N=384, m=10, prec="f32", sites=64),
        # one FP64 application on a p = 5 slab with projectors, a width that no tile divides
        _case("slab-p5-hx-ragged", "hx", 5, (20, 20, 40), N=200, sites=64),
        # a k-point of the p = 4 slab: complex vectors
        _case("slab-p4-bloch", "bloch", 4, (24, 24, 48), N=128, m=10, kx=0.5 * math.pi / 24, ky=0.25 * math.pi / 24),
        # gradients of a filtered loss in X, V and E on the p = 6 slab (forward, reverse sweep)
        _case("slab-p6-gradient", "grad", 6, (16, 16, 32), N=32, m=20),
        # low degree on a fine mesh with a few vectors more than a multiple of 16
        _case("slab-p2-filter", "filter", 2, (30, 30, 60), N=100, m=12),
        # an odd mesh, odd width and odd leading dimension, periodic along all axes
        _case("odd-p4-hx", "hx", 4, (7, 5, 9), N=33, bc="PPP", pad=2),
        # the field response of a slab: bounds, two subspace iterations, density, planar average, dipole
        _case("slab-p4-response", "response", 4, (12, 12, 24), N=64, m=12),
        # electrostatics of the constant-field setup: conjugate gradients on the wavefunction mesh
        _case("slab-p4-poisson", "poisson", 4, (24, 24, 48), bc="PPN"),
        # spectrum bounds: single-vector products and reorthogonalisation
        _case("slab-p4-bounds", "bounds", 4, (24, 24, 48)),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the ranges above: degrees 1 to 7, a few cells to the slabs' 24 x 24 x 48, 1 to 256 vectors."""
    kind = rng.choice(["filter"] * 8 + ["hx"] * 3 + ["bloch"] * 2 + ["grad"] * 2 + ["f32"] * 2 + ["poisson", "bounds", "response"])
    prec = "f64"
    if kind == "f32":
        kind, prec = "filter", "f32"
    while True:
        p = rng.choice([1, 2, 3, 3, 4, 4, 4, 5, 5, 6, 6, 7])
        bc = rng.choice(["PPD"] * 5 + ["DDD", "PPP"])
        cells = (_log(rng, 3, 24), _log(rng, 3, 24), _log(rng, 3, 48))
        N, m, pad, sites, kx, ky = _log(rng, 1, 256), rng.randint(4, 30), 0, 0, 0.0, 0.0
        if kind == "hx":
            m, pad = 1, rng.choice([0, 0, 1, 2, 6])
        if kind in ("filter", "hx") and min(cells) >= 6 and rng.random() < 0.3:
            sites = rng.randint(1, 32)
        if kind == "bloch":
            bc, N, m = "PPD", max(1, N // 2), max(4, m // 2)
            kx, ky = round(rng.uniform(0.05, 1.0), 4), round(rng.uniform(0.0, 1.0), 4)
        if kind == "grad":
            N, m = max(1, N // 4), max(4, m // 2)
        if kind == "poisson":
            N, m, bc = 1, 1, rng.choice(["PPN", "PPN", "DDD"])
        if kind == "bounds":
            N, m = 1, 1
        if kind == "response":
            N, m, bc = max(8, N // 4), rng.randint(8, 16), "PPD"
        n = 1
        for c, b in zip(cells, bc):
            n *= c * p + {"D": -1, "P": 0, "N": 1}[b]
        dense = (p + 1) ** 6 * cells[0] * cells[1] * cells[2] * N * m * {"bloch": 4, "grad": 3}.get(kind, 1)
        blocks = m + 6 if kind == "grad" else 6 if kind == "bloch" else 3
        if n < 200 or n > 2_000_000 or 8 * N > n or dense > 0.25 * 5 ** 6 * 27648 * 256 * 30 or n * N * 8 * blocks > 8e9:
            continue
        return _case(None, kind, p, cells, N, m, bc, prec, pad, sites, kx, ky)


# ------------------------------------------------------------------- inputs

def _gll(p):
    """GLL nodes and weights on [-1, 1]."""
    c = np.zeros(p + 1)
    c[p] = 1.0
    x = np.concatenate([[-1.0], np.sort(np.polynomial.legendre.legroots(np.polynomial.legendre.legder(c)).real), [1.0]])
    for _ in range(3):  # Newton on (1 - x^2) P_p'
        d1 = np.polynomial.legendre.legval(x[1:-1], np.polynomial.legendre.legder(c))
        d2 = np.polynomial.legendre.legval(x[1:-1], np.polynomial.legendre.legder(c, 2))
        x[1:-1] -= d1 / d2
    w = 2.0 / (p * (p + 1) * np.polynomial.legendre.legval(x, c) ** 2)
    return x, w


def _axis(ncell, p, bc):
    """One axis of cells of edge 1: coordinates and lumped masses of the free
    nodes, the assembled stiffness, consistent mass and advection matrices,
    and the free index of each cell's local nodes (-1: a Dirichlet node)."""
    x, w = _gll(p)
    y, wy = np.polynomial.legendre.leggauss(p + 2)
    V = np.vander(x, p + 1, increasing=True)
    coef = np.linalg.inv(V)                      # basis j = sum_k coef[k, j] t^k
    val = np.vander(y, p + 1, increasing=True) @ coef
    der = (np.vander(y, p + 1, increasing=True)[:, :-1] * np.arange(1, p + 1)) @ coef[1:]
    k1, m1, g1 = 2.0 * der.T @ (wy[:, None] * der), 0.5 * val.T @ (wy[:, None] * val), val.T @ (wy[:, None] * der)
    K = ncell * p
    nf = K + {"D": -1, "P": 0, "N": 1}[bc]
    free = lambda g: (-1 if g in (0, K) else g - 1) if bc == "D" else g % K if bc == "P" else g  # noqa: E731
    out = {"K": np.zeros((nf, nf)), "M": np.zeros((nf, nf)), "G": np.zeros((nf, nf)), "mass": np.zeros(nf),
           "x": np.zeros(nf), "idx": np.array([[free(c * p + i) for i in range(p + 1)] for c in range(ncell)])}
    for c in range(ncell):
        f = out["idx"][c]
        ok = f >= 0
        at = np.ix_(f[ok], f[ok])
        for name, a in (("K", k1), ("M", m1), ("G", g1)):
            np.add.at(out[name], at, a[np.ix_(ok, ok)])
        np.add.at(out["mass"], f[ok], 0.5 * w[ok])
        out["x"][f[ok]] = c + 0.5 * (x[ok] + 1.0)
    if bc == "P":
        out["x"][0] = 0.0
    out["pts"] = np.add.outer(np.arange(ncell), 0.5 * (x + 1.0))
    out["w"] = 0.5 * w
    return out


def _axes(c):
    return [_axis(c["n" + a], c["p"], b) for a, b in zip("xyz", c["bc"])]


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _generator(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * stream + seed)
    return g


def _sites(c, seed, spacing=3.0):
    """Well centres: a lattice in the middle third of the box, each moved a little at random."""
    L = [c["nx"], c["ny"], c["nz"]]
    lo = [0.0, 0.0, L[2] / 3.0]
    span = [L[0], L[1], L[2] / 3.0]
    cnt = [max(1, min(8, int(s / spacing))) for s in span]
    r = np.random.default_rng([seed, 1])
    grid = np.array([[lo[a] + span[a] * (i[a] + 0.5) / cnt[a] for a in range(3)] for i in np.ndindex(*cnt)])
    return grid + r.uniform(-0.3, 0.3, grid.shape)


def _wells(c, seed, pts):
    """Gaussian wells at the tensor product of per-axis points: (nz, ny, nx)."""
    gs = []
    for a, ax in enumerate("xyz"):
        d = np.subtract.outer(_sites(c, seed)[:, a], pts[a])
        if c["bc"][a] == "P":
            d -= c["n" + ax] * np.round(d / c["n" + ax])
        gs.append(_t(np.exp(-d * d / (2 * SIGMA * SIGMA))))
    out = torch.zeros(len(pts[2]), len(pts[1]), len(pts[0]), dtype=F64, device=DEV)
    for x, y, z in zip(*gs):
        out += z[:, None, None] * y[None, :, None] * x[None, None, :]
    return out


def _potential(c, seed, axes):
    """V at the cell GLL points, (cells, (p+1)^3), x fastest."""
    n1 = c["p"] + 1
    V = DEPTH * _wells(c, seed, [a["pts"].reshape(-1) for a in axes])
    V = V.view(c["nz"], n1, c["ny"], n1, c["nx"], n1).permute(0, 2, 4, 1, 3, 5)
    return V.reshape(-1, n1 ** 3).contiguous()


def _field(c):
    """(E, z0): the linear field is left out where z is periodic."""
    return (0.0 if c["bc"][2] == "P" else FIELD), 0.5 * c["nz"]


def _bounds(c, axes):
    """An upper bound b of the spectrum from the per-axis matrices, a lower
    scaling point a0 and the cut a (fixed numbers, as a program keeps them)."""
    b = 0.0
    k, m = [], []
    for a in axes:
        d = a["mass"] ** -0.5
        k.append(np.linalg.eigvalsh(0.5 * d[:, None] * a["K"] * d)[-1])
        m.append(np.linalg.eigvalsh(d[:, None] * a["M"] * d)[-1])
    b = k[0] * m[1] * m[2] + m[0] * k[1] * m[2] + m[0] * m[1] * k[2] + 1.0
    b += 0.5 * (c["kx"] ** 2 + c["ky"] ** 2) + (1.0 + c["kx"] + c["ky"]) * (c["kind"] == "bloch")
    b += 2.0 * (c["sites"] > 0)
    n = math.prod(len(a["x"]) for a in axes)
    a0 = -1.5
    return a0 + (b - a0) * (c["N"] / n) ** (2.0 / 3.0), float(b), a0


def _projector_sites(c, seed):
    r = np.random.default_rng([seed, 2])
    L = np.array([c["nx"], c["ny"], c["nz"]], dtype=float)
    return r.uniform(0.1, 0.9, (c["sites"], 3)) * L, r.uniform(-1.0, 1.0, (c["sites"], 9))


def _block(c, n, seed, stream=3):
    """The wavefunction block, i.i.d. N(0,1); complex for the Bloch kind; a view of a wider buffer where pad > 0."""
    cols = c["N"] + c["pad"]
    if c["kind"] == "bloch":
        return torch.view_as_complex(torch.randn(n, cols, 2, generator=_generator(seed, stream), dtype=F64, device=DEV))
    return torch.randn(n, cols, generator=_generator(seed, stream), dtype=F64, device=DEV)[:, :c["N"]]


def _charge(c, seed, axes):
    return _wells(c, seed, [a["x"] for a in axes]).reshape(-1)


# ---------------------------------------------------------------- the passes

def prepare(case, seed):
    c, axes = case, _axes(case)
    mesh = fe.Mesh([c["nx"], c["ny"], c["nz"]], [c["nx"], c["ny"], c["nz"]], c["p"], [BC[b] for b in c["bc"]])
    E, z0 = _field(c)
    s = {"c": c, "mesh": mesh, "E": E, "z0": z0}
    if c["kind"] == "poisson":
        s["charge"] = _charge(c, seed, axes)
        s["phi"] = torch.empty_like(s["charge"])
        return s
    s["V"] = _potential(c, seed, axes)
    s["bounds"] = _bounds(c, axes)
    if c["sites"]:
        mesh.set_nonlocal(*_projector_sites(c, seed), R_CUT, R_G)
    if c["kind"] in ("bounds", "response"):
        s["v0"] = torch.randn(mesh.n, generator=_generator(seed, 4), dtype=F64, device=DEV)
    if c["kind"] == "bounds":
        mesh.set_potential(s["V"], E, z0)
        return s
    s["X"] = _block(c, mesh.n, seed)
    if c["kind"] == "hx":
        mesh.set_potential(s["V"], E, z0)
        s["Y"] = torch.empty(mesh.n, c["N"] + c["pad"], dtype=F64, device=DEV)[:, :c["N"]]
    if c["kind"] in ("filter", "bloch"):
        s["Y"] = torch.empty_like(s["X"])
        s["work"] = torch.empty(mesh.n * c["N"] * (2 if c["kind"] == "bloch" else 1), dtype=F64, device=DEV)
    if c["kind"] == "bloch":
        mesh.set_kpoint(c["kx"], c["ky"])
    if c["kind"] == "grad":
        s["X"].requires_grad_(True)
        s["V"].requires_grad_(True)
        s["Et"] = torch.tensor(E, dtype=F64, device=DEV, requires_grad=True)
        s["w"] = torch.rand(c["N"], generator=_generator(seed, 5), dtype=F64, device=DEV)
    if c["kind"] == "response":
        s["f"] = torch.ones(c["N"], dtype=F64, device=DEV)
    return s


def run(s):
    c, mesh, E, z0 = s["c"], s["mesh"], s["E"], s["z0"]
    kind = c["kind"]
    if kind == "hx":
        return mesh.hx(s["X"], s["Y"], prec=c["prec"])
    if kind == "filter":
        mesh.set_potential(s["V"], E, z0)
        return mesh.cheb_filter(s["X"], c["m"], *s["bounds"], prec=c["prec"], Y=s["Y"], work=s["work"])
    if kind == "bloch":
        mesh.set_potential(s["V"], E, z0)
        return mesh.cheb_filter_k(s["X"], c["m"], *s["bounds"], Y=s["Y"], work=s["work"])
    if kind == "grad":
        a, b, a0 = s["bounds"]
        Y = fe.cheb_filter(s["X"], s["V"], s["Et"], mesh, c["m"], a, b, a0, z0=z0)
        loss = (s["w"] * (s["X"] * Y).sum(0)).sum()
        gX, gV, gE = torch.autograd.grad(loss, (s["X"], s["V"], s["Et"]))
        return {"loss": loss.detach(), "X": gX, "V": gV, "E": gE}
    if kind == "bounds":
        return list(mesh.lanczos_bounds(s["v0"], 10))
    if kind == "response":
        mesh.set_potential(s["V"], E, z0)
        a0, b = mesh.lanczos_bounds(s["v0"], 10)
        a = solver.weyl_cut(a0, b, c["N"], mesh.n)
        hist, X = solver.subspace_iteration(mesh, s["X"], c["m"], 2, a, b, a0)
        rho = mesh.density(X, s["f"])
        return {"theta": hist[-1], "rho": rho, "planar": mesh.planar_average(rho), "mu": mesh.dipole(rho, z0)}
    phi, _, _ = mesh.poisson(s["charge"], tol=1e-12, phi=s["phi"])
    return phi


# ------------------------------------------------------------------ the work

def work(case):
    """The recurrence's own traffic and arithmetic: per step and value the two
    blocks that are read and the one that is written (24 bytes; 16 for a
    product), and the per-axis contractions of the tensor-product stiffness
    (p + 2 products per value on the average of an axis' nodes; seven
    contractions for K, ten with the k.G term of complex vectors)."""
    c, p = case, case["p"]
    n = math.prod(c["n" + a] * p + {"D": -1, "P": 0, "N": 1}[b] for a, b in zip("xyz", c["bc"]))
    per = 14 * (p + 2) + 8
    nN = n * c["N"]
    nl = 0.0
    if c["sites"]:
        nl = c["sites"] * 4.0 / 3.0 * math.pi * R_CUT ** 3 * p ** 3 * c["N"]  # support entries x vectors
    m = c["m"]
    if c["kind"] == "hx":
        return {"bytes": 16 * nN + 8 * n + 24 * nl, "flops": per * nN + 36 * nl}
    if c["kind"] == "filter":
        return {"bytes": 16 * nN + 24 * nN * (m - 1) + 8 * n * m + 24 * nl * m, "flops": (per * nN + 36 * nl) * m}
    if c["kind"] == "bloch":
        return {"bytes": 2 * (16 + 24 * (m - 1)) * nN + 8 * n * m, "flops": 2 * (20 * (p + 2) + 8) * nN * m}
    if c["kind"] == "grad":  # forward, the reverse sweep, and Y_k read once more for the dots with the adjoint
        return {"bytes": (24 + 32) * nN * m, "flops": (2 * per + 2) * nN * m}
    if c["kind"] == "bounds":  # k products, twice V (V^T w) per step
        k = 10
        return {"bytes": 16.0 * n * k + 8 * n * 2 * k * (k + 1), "flops": per * n * k + 4 * n * k * (k + 1)}
    if c["kind"] == "response":
        bounds = work(dict(c, kind="bounds", N=1))
        filt = work(dict(c, kind="filter"))
        dense = 8.0 * n * c["N"] ** 2
        return {"bytes": bounds["bytes"] + 2 * (filt["bytes"] + 112 * nN) + 8 * nN + 24 * n,
                "flops": bounds["flops"] + 2 * (filt["flops"] + dense + per * nN) + 3 * nN}
    its = 5.0 * p * max(c["nx"], c["ny"], c["nz"])  # about; eight vector passes an iteration
    return {"bytes": 64 * n * its, "flops": (per + 14) * n * its}


# ------------------------------------------------------- the same in 64 bits

class _Operator:
    """H~ from dense one-dimensional matrices, in torch."""

    def __init__(self, c, seed):
        self.c, self.axes = c, _axes(c)
        self.shape = [len(a["x"]) for a in self.axes][::-1]
        self.n = math.prod(self.shape)
        d = [a["mass"] ** -0.5 for a in self.axes]
        self.K = [_t(0.5 * d[i][:, None] * a["K"] * d[i]) for i, a in enumerate(self.axes)]
        self.M = [_t(d[i][:, None] * a["M"] * d[i]) for i, a in enumerate(self.axes)]
        self.G = [_t(d[i][:, None] * a["G"] * d[i]) for i, a in enumerate(self.axes)]
        mx, my, mz = (_t(a["mass"]) for a in self.axes)
        self.mass = (mz[:, None, None] * my[None, :, None] * mx[None, None, :]).reshape(-1)
        self.z = _t(self.axes[2]["x"])[:, None, None].expand(self.shape).reshape(-1)
        self.E, self.z0 = _field(c)
        self.C = None
        if c["kind"] != "poisson":
            V = DEPTH * _wells(c, seed, [a["x"] for a in self.axes]).reshape(-1)
            self.v = V - self.E * (self.z - self.z0)
            if c["sites"]:
                self._projectors(seed)

    def _projectors(self, seed):
        cen, D = _projector_sites(self.c, seed)
        X = [_t(a["x"]) for a in self.axes]
        self.C = []
        for R, Ds in zip(cen, D):
            d = []
            for a, ax in enumerate("xyz"):
                e = X[a] - R[a]
                if self.c["bc"][a] == "P":
                    e = e - self.c["n" + ax] * torch.round(e / self.c["n" + ax])
                d.append(e)
            r2 = d[2][:, None, None] ** 2 + d[1][None, :, None] ** 2 + d[0][None, None, :] ** 2
            at = (r2.reshape(-1) < R_CUT * R_CUT).nonzero()[:, 0]
            x, y = d[0][at % self.shape[2]], d[1][(at // self.shape[2]) % self.shape[1]]
            z = d[2][at // (self.shape[2] * self.shape[1])]
            S = torch.stack([torch.ones_like(x), x, y, z, x * y, y * z, z * x, x * x - y * y,
                             2 * z * z - x * x - y * y], 1)
            P = S * torch.exp(-(x * x + y * y + z * z) / (2 * R_G * R_G))[:, None] * self.mass[at].sqrt()[:, None]
            self.C.append((at, P / P.norm(dim=0), _t(Ds)))

    def _along(self, A, a, X):
        """A along axis a (0: x) of X (nz, ny, nx, N)."""
        nz, ny, nx, N = X.shape
        if a == 0:
            return torch.matmul(A, X.view(nz * ny, nx, N)).view(X.shape)
        if a == 1:
            return torch.matmul(A, X.view(nz, ny, nx * N)).view(X.shape)
        return torch.matmul(A, X.view(nz, ny * nx * N)).view(X.shape)

    def real(self, X):
        """H~ X for a contiguous (n, N) block."""
        U = X.view(*self.shape, X.shape[1])
        MX, KX = self._along(self.M[0], 0, U), self._along(self.K[0], 0, U)
        B = self._along(self.M[1], 1, KX)
        del KX
        B += self._along(self.K[1], 1, MX)
        A = self._along(self.M[1], 1, MX)
        del MX
        out = self._along(self.M[2], 2, B)
        del B
        out += self._along(self.K[2], 2, A)
        del A
        out = out.view(X.shape)
        out.addcmul_(X, self.v[:, None].expand_as(X))
        for at, P, D in self.C or ():
            out.index_add_(0, at, P @ (D[:, None] * (P.T.contiguous() @ X[at])))
        return out

    def kg(self, X):
        """M^-1/2 (k.G) M^-1/2 X."""
        U = X.view(*self.shape, X.shape[1])
        MX, GX = self._along(self.M[0], 0, U), self._along(self.G[0], 0, U)
        B = self.c["kx"] * self._along(self.M[1], 1, GX) + self.c["ky"] * self._along(self.G[1], 1, MX)
        return self._along(self.M[2], 2, B).view(X.shape)

    def apply(self, X):
        """X: (re, im) for the Bloch kind, else one block."""
        if self.c["kind"] != "bloch":
            return self.real(X)
        kk = 0.5 * (self.c["kx"] ** 2 + self.c["ky"] ** 2)
        re, im = X
        return (self.real(re) + kk * re + self.kg(im), self.real(im) + kk * im - self.kg(re))


def _coefficients(m, a, b, a0):
    e, c = 0.5 * (b - a), 0.5 * (b + a)
    s1 = s = e / (a0 - c)
    al, be = [s1 / e], [0.0]
    for _ in range(1, m):
        sn = 1.0 / (2.0 / s1 - s)
        al.append(2.0 * sn / e)
        be.append(s * sn)
        s = sn
    return al, be, c


def _lin(f, *blocks):
    """f over blocks or over their (re, im) pairs."""
    return tuple(f(*p) for p in zip(*blocks)) if isinstance(blocks[0], tuple) else f(*blocks)


def _filter(op, X, m, a, b, a0, keep=False):
    al, be, c = _coefficients(m, a, b, a0)
    Ys = [X]
    for k in range(m):
        H = op.apply(Ys[-1])
        Y = _lin(lambda h, y: al[k] * (h - c * y), H, Ys[-1])
        if k:
            Y = _lin(lambda y, o: y.sub_(o, alpha=be[k]), Y, Ys[-2])
        Ys.append(Y)
        if not keep:
            Ys = Ys[-2:]
    return Ys if keep else Ys[-1]


def _lanczos(op, v, k=10):
    V, al, be = [v / v.norm()], [], []
    for j in range(k):
        w = op.real(V[-1][:, None].contiguous())[:, 0]
        al.append(float(V[-1] @ w))
        for _ in range(2):
            Q = torch.stack(V, 1)
            w = w - Q @ (Q.T @ w)
        be.append(float(w.norm()))
        V.append(w / be[-1])
    T = np.diag(al) + np.diag(be[:-1], 1) + np.diag(be[:-1], -1)
    ev = np.linalg.eigvalsh(T)
    return float(ev[0]), float(ev[-1] + abs(be[-1]))


def _poisson(op, c, seed):
    """K phi = 4 pi M s by the joint eigenvectors of each axis' stiffness and consistent mass."""
    lam, W = [], []
    for a in op.axes:
        L = np.linalg.inv(np.linalg.cholesky(a["M"]))
        e, q = np.linalg.eigh(L @ a["K"] @ L.T)
        lam.append(_t(e))
        W.append(_t(L.T @ q))
    b = 4.0 * math.pi * op.mass * _charge(c, seed, op.axes)
    singular = "D" not in c["bc"]
    if singular:
        b = b - op.mass * (b.sum() / op.mass.sum())
    u = b.view(*op.shape, 1)
    for a in range(3):
        u = op._along(W[a].T.contiguous(), a, u.contiguous())
    den = lam[2][:, None, None] + lam[1][None, :, None] + lam[0][None, None, :]
    if singular:
        den[0, 0, 0] = math.inf
    u = u / den[..., None]
    for a in range(3):
        u = op._along(W[a], a, u.contiguous())
    phi = u.reshape(-1)
    return phi - (op.mass @ phi) / op.mass.sum() if singular else phi


def exact(case, seed):
    c = case
    op = _Operator(c, seed)
    bounds = None if c["kind"] == "poisson" else _bounds(c, op.axes)
    if c["kind"] == "poisson":
        return _poisson(op, c, seed)
    if c["kind"] == "bounds":
        return list(_lanczos(op, torch.randn(op.n, generator=_generator(seed, 4), dtype=F64, device=DEV)))
    X = _block(c, op.n, seed)
    if c["kind"] == "hx":
        return op.apply(X.contiguous())
    if c["kind"] == "filter":
        return _filter(op, X.contiguous(), c["m"], *bounds)
    if c["kind"] == "bloch":
        return torch.complex(*_filter(op, (X.real.contiguous(), X.imag.contiguous()), c["m"], *bounds))
    if c["kind"] == "response":
        a0, b = _lanczos(op, torch.randn(op.n, generator=_generator(seed, 4), dtype=F64, device=DEV))
        a = a0 + (b - a0) * (c["N"] / op.n) ** (2.0 / 3.0)
        for _ in range(2):
            Q, _ = torch.linalg.qr(_filter(op, X.contiguous(), c["m"], a, b, a0))
            H = Q.T @ op.apply(Q.contiguous())
            theta, W = torch.linalg.eigh(0.5 * (H + H.T))
            X = Q @ W
            a, a0 = float(theta[-1]), float(theta[0])
        rho = 2.0 * (X * X).sum(1) / op.mass
        mx, my, mz = (_t(a["mass"]) for a in op.axes)
        planar = torch.einsum("kji,j,i->k", rho.view(op.shape), my, mx)
        mu = (planar * mz * (_t(op.axes[2]["x"]) - op.z0)).sum()
        return {"theta": theta.cpu().numpy(), "rho": rho, "planar": planar, "mu": float(mu)}
    # grad: loss = sum_i w_i <x_i, T(H~) x_i>; dL/dX = 2 T(H~) X w, and the
    # reverse sweep for the derivative in the diagonal potential
    w = torch.rand(c["N"], generator=_generator(seed, 5), dtype=F64, device=DEV)
    Ys = _filter(op, X, c["m"], *bounds, keep=True)
    al, be, cc = _coefficients(c["m"], *bounds)
    loss = (w * (X * Ys[-1]).sum(0)).sum()
    g = torch.zeros(op.n, dtype=F64, device=DEV)
    nxt, cur = None, X * w
    for k in range(c["m"] - 1, -1, -1):
        g += al[k] * (cur * Ys[k]).sum(1)
        new = al[k] * (op.apply(cur) - cc * cur)
        if nxt is not None:
            new -= be[k + 1] * nxt
        nxt, cur = cur, new
    # shape factors |J| w_q / M_I of each cell point, zero at Dirichlet nodes
    n1 = c["p"] + 1
    gm = torch.cat([g / op.mass, torch.zeros(1, dtype=F64, device=DEV)])
    ix, iy, iz = (_t(a["idx"].reshape(-1)) for a in op.axes)
    wx, wy, wz = (_t(np.tile(a["w"], len(a["idx"]))) for a in op.axes)
    at = ix[None, None, :] + op.shape[2] * (iy[None, :, None] + op.shape[1] * iz[:, None, None])
    at[(ix < 0)[None, None, :].expand_as(at) | (iy < 0)[None, :, None].expand_as(at) | (iz < 0)[:, None, None].expand_as(at)] = op.n
    gV = gm[at] * (wz[:, None, None] * wy[None, :, None] * wx[None, None, :])
    gV = gV.view(c["nz"], n1, c["ny"], n1, c["nx"], n1).permute(0, 2, 4, 1, 3, 5).reshape(-1, n1 ** 3)
    return {"loss": loss, "X": 2.0 * Ys[-1] * w, "V": gV.contiguous(), "E": -(g * (op.z - op.z0)).sum()}
