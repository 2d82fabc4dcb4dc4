"""The work that users of the spectral-element Poisson engine have it do, as
measurable cases.

Every case goes through the public Python entry points (``Mesh``, ``Batch``,
``Projection``).  A case is a dict of plain values; its ``kind`` says what one
pass is:

  apply       w = mask(Q Q^T A_L u): the assembled operator on a resident mesh
              (a time-stepper's residual, a user's own Krylov method)
  iterate     a fixed number of FP64 Jacobi-PCG iterations (the headline step)
  solve       a whole solve to 1e-10, FP64 or mixed, Jacobi or with the coarse
              term of Eq. 6
  precond     z = M^-1 r with the Schwarz local solves and / or the coarse term
  batch       many boxes of mixed orders and sizes solved together
  projection  a time-stepper's projection space: a few solutions join the
              basis, the next right-hand side is formed and projected

``exact`` gives the same results in 64 bits from the mathematics alone (GLL
collocation, isoparametric hexahedra, lexicographic numbering), in plain torch
and numpy.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2109_03592_amd as sem

F64 = torch.float64


# ---------------------------------------------------------------------------
# the cases
def listed():
    return [
        # the smallest call: one apply on a 64-element jittered test box, bound by launches
        {"name": "apply_box_n5_tiny", "kind": "apply", "N": 5, "nx": 4, "ny": 4, "nz": 4, "map": "box",
         "per": 0, "dtype": "f64", "helm": False},
        # low order on an odd-sized box periodic in x and y (the N-sweep's 16,250 elements)
        {"name": "apply_box_n3_periodic", "kind": "apply", "N": 3, "nx": 25, "ny": 26, "nz": 25, "map": "box",
         "per": 3, "dtype": "f64", "helm": False},
        # the headline workload: the pipe at one GPU's share, 221,184 elements
        {"name": "apply_pipe_n7", "kind": "apply", "N": 7, "nx": 48, "ny": 48, "nz": 96, "map": "pipe",
         "per": 4, "dtype": "f64", "helm": False},
        # the same operator in FP32 on the pipe of the time-stepping workload
        {"name": "apply_pipe_n7_f32", "kind": "apply", "N": 7, "nx": 24, "ny": 24, "nz": 48, "map": "pipe",
         "per": 4, "dtype": "f32", "helm": False},
        # the higher production order, in the Helmholtz form of a velocity solve
        {"name": "apply_box_n9_helmholtz", "kind": "apply", "N": 9, "nx": 23, "ny": 24, "nz": 25, "map": "box",
         "per": 0, "dtype": "f64", "helm": True},
        # Jacobi-PCG iterations, the benchmark's step
        {"name": "iterate_pipe_n7", "kind": "iterate", "N": 7, "nx": 32, "ny": 32, "nz": 64, "map": "pipe",
         "per": 4, "iters": 32},
        # a small whole solve, bound by the latency of an iteration
        {"name": "solve_box_n7_small", "kind": "solve", "N": 7, "nx": 4, "ny": 4, "nz": 4, "map": "box", "per": 0,
         "precision": "fp64", "coarse": 0},
        # a mixed-precision solve on the pipe slab the accuracy figures are quoted on
        {"name": "solve_slab_mixed", "kind": "solve", "N": 7, "nx": 12, "ny": 12, "nz": 8, "map": "pipe", "per": 4,
         "precision": "mixed", "coarse": 0},
        # the recommended preconditioner: Jacobi + coarse term, four Chebyshev steps
        {"name": "solve_pipe_coarse", "kind": "solve", "N": 7, "nx": 16, "ny": 16, "nz": 16, "map": "pipe", "per": 4,
         "precision": "fp64", "coarse": 4},
        # both parts of Eq. 6's preconditioner, applied in a user's own Krylov method
        {"name": "precond_pipe_schwarz", "kind": "precond", "N": 7, "nx": 24, "ny": 24, "nz": 48, "map": "pipe",
         "per": 4, "schwarz": True, "coarse": 4},
        # many boxes at once, the coarse term on those of 512 elements and more (the serving setting)
        {"name": "batch_boxes", "kind": "batch", "count": 12, "emin": 8, "emax": 1024, "orders": "5,7,9", "shape": 100,
         "precision": "fp64", "coarse_min": 512},
        # a time step's bookkeeping: six solutions join the basis, the next right-hand side is projected
        {"name": "projection_pipe_n7", "kind": "projection", "N": 7, "nx": 24, "ny": 24, "nz": 24, "map": "pipe",
         "per": 4, "vectors": 6},
    ]


def _spread(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_mesh(rng, orders, lo, hi):
    """A mesh of `lo` to `hi` local points: order, element counts (odd ones
    among them), mapping and periodic axes."""
    N = rng.choice(orders)
    E = max(8.0, _spread(rng, lo, hi) / (N + 1) ** 3)
    edge = E ** (1.0 / 3.0)
    nx = max(2, int(round(edge * rng.uniform(0.7, 1.3))))
    ny = max(2, int(round(edge * rng.uniform(0.7, 1.3))))
    nz = max(2, int(round(E / (nx * ny))))
    pipe = rng.random() < 0.5
    return {"N": N, "nx": nx, "ny": ny, "nz": nz, "map": "pipe" if pipe else "box",
            "per": 4 if pipe else rng.choice([0, 0, 1, 2, 3, 4, 5])}


def draw(rng):
    kind = rng.choice(["apply"] * 5 + ["iterate"] + ["solve"] * 2 + ["precond", "batch", "projection"])
    if kind == "apply":
        # every order the engine is built for, from a few thousand to tens of millions of points
        c = _draw_mesh(rng, list(range(2, 13)) + [5, 7, 7, 9, 14, 17], 4e3, 3e7)
        c["dtype"] = rng.choice(["f64", "f64", "f32"])
        c["helm"] = rng.random() < 0.25
    elif kind == "iterate":
        c = _draw_mesh(rng, [3, 4, 5, 6, 7, 8, 9, 10, 12], 1e4, 2e7)
        c["iters"] = rng.choice([16, 24, 32])
    elif kind == "solve":
        c = _draw_mesh(rng, [3, 5, 7, 9], 5e3, 1e6)
        c["precision"] = rng.choice(["fp64", "mixed"])
        c["coarse"] = rng.choice([0, 4])
    elif kind == "precond":
        c = _draw_mesh(rng, [3, 4, 5, 6, 7, 8, 9], 2e4, 1e7)
        c["schwarz"] = rng.random() < 0.7
        c["coarse"] = rng.choice([2, 4, 8])
    elif kind == "batch":
        c = {"count": rng.randint(3, 12), "emin": 8, "emax": rng.choice([64, 256, 768]), "orders": "5,7,9",
             "shape": rng.randrange(100, 1000), "precision": rng.choice(["fp64", "mixed"]), "coarse_min": 512}
    else:
        c = _draw_mesh(rng, [4, 5, 6, 7, 8, 9], 2e4, 7e6)
        c["vectors"] = rng.randint(2, 8)
    c["kind"] = kind
    return c


# ---------------------------------------------------------------------------
# inputs: the same numbers for the engine and for exact()
def _nel(case):
    return (case["nx"], case["ny"], case["nz"])


def _periodic(case):
    return tuple((case["per"] >> d) & 1 for d in range(3))


def _vertices(nel, seed, amp=0.05):
    """Unit-box vertex lattice, interior vertices moved by up to 5% of an element."""
    nx, ny, nz = nel
    rng = np.random.default_rng(seed)
    z, y, x = np.meshgrid(np.arange(nz + 1), np.arange(ny + 1), np.arange(nx + 1), indexing="ij")
    h = np.array([1.0 / nx, 1.0 / ny, 1.0 / nz])
    V = np.stack([x, y, z], axis=-1).reshape(-1, 3) * h
    inner = ((x > 0) & (x < nx) & (y > 0) & (y < ny) & (z > 0) & (z < nz)).reshape(-1)
    V[inner] += (rng.uniform(-amp, amp, size=V.shape) * h)[inner]
    return np.ascontiguousarray(V)


def _random(n, seed, lo=-1.0, hi=1.0):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return torch.rand(int(n), generator=g, dtype=F64, device="cuda") * (hi - lo) + lo


def _rhs_values(n, seed):
    """One U[-1, 1) value per global node, mean removed."""
    v = _random(n, seed)
    return v - v.mean()


def _smooth_values(ref, seed, count):
    """`count` successive solutions of a time-stepping run, one value per
    global node: a travelling wave with a little roughness of its own."""
    x, y, z = ref.global_coords()
    out = []
    for m in range(count):
        v = torch.sin(math.pi * (x + 0.15 * m)) * torch.cos(math.pi * y * (1 + 0.05 * m)) * torch.cos(0.6 * z)
        out.append(v + 0.02 * _random(v.numel(), 1000 * seed + m))
    return out


def _mesh(case, seed, fp32=False):
    if case["map"] == "pipe":
        return sem.pipe_mesh(*_nel(case), N=case["N"], length=10.0, with_fp32=fp32)
    return sem.box_mesh(case["N"], _nel(case), vertices=_vertices(_nel(case), seed), periodic=_periodic(case),
                        with_fp32=fp32)



def _boxes(case, seed):
    """The meshes of a batch as (N, nel, vertex seed): element counts from a
    log-uniform target."""
    out = []
    for q in range(case["count"]):
        rng = np.random.default_rng(case["shape"] + q)
        e = math.exp(rng.uniform(math.log(case["emin"]), math.log(case["emax"])))
        N = int(rng.choice([int(s) for s in case["orders"].split(",")]))
        nx = max(1, round(e ** (1 / 3)))
        ny = max(1, round(math.sqrt(e / nx)))
        out.append((N, (nx, ny, max(1, round(e / (nx * ny)))), seed + q))
    return out


def _box_case(N, nel):
    return {"N": N, "nx": nel[0], "ny": nel[1], "nz": nel[2], "map": "box", "per": 0}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        meshes, bs = [], []
        for N, nel, vs in _boxes(case, seed):
            m = _mesh(_box_case(N, nel), vs, case["precision"] == "mixed")
            if m.E >= case["coarse_min"]:
                m.set_coarse(4, 0.05)
            meshes.append(m)
            bs.append(m.scatter(_rhs_values(m.n_global, vs)))
        return {"case": case, "meshes": meshes, "b": bs, "batch": sem.Batch(max_slots=case["count"])}
    fp32 = case.get("dtype") == "f32" or case.get("precision") == "mixed"
    m = _mesh(case, seed, fp32)
    s = {"case": case, "mesh": m}
    if kind == "apply":
        if case["helm"]:
            m.set_helmholtz(_random(m.n_local, seed + 1, 0.5, 2.0), _random(m.n_local, seed + 2, 0.0, 3.0))
        s["u"] = m.scatter(_random(m.n_global, seed))
        if fp32:
            s["u"] = s["u"].float()
        s["w"] = torch.empty_like(s["u"])
    elif kind in ("iterate", "solve", "precond"):
        if case.get("schwarz"):
            m.set_schwarz(True)
        if case.get("coarse"):
            m.set_coarse(case["coarse"], 0.05)
        s["b"] = m.scatter(_rhs_values(m.n_global, seed))
        s["z"] = m.empty()
    else:
        s["f"] = _random(m.n_local, seed)
        s["xs"] = [m.scatter(v) for v in _smooth_values(_Ref(case, seed), seed, case["vectors"])]
        s["proj"] = sem.Projection(m, 8)
        s["b"], s["z"] = m.empty(), m.empty()
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "apply":
        return s["mesh"].axgs(s["u"], s["w"])
    if kind == "iterate":
        x, _ = s["mesh"].solve(s["b"], fixed_iters=c["iters"])
        return x
    if kind == "solve":
        x, _ = s["mesh"].solve(s["b"], tol=1e-10, max_iter=20000, precision=c["precision"])
        return x
    if kind == "precond":
        return s["mesh"].precond(s["b"], s["z"])
    if kind == "batch":
        xs, _ = s["batch"].solve(s["meshes"], s["b"], tol=1e-10, max_iter=20000, precision=c["precision"])
        return xs
    s["proj"].reset()
    for x in s["xs"]:
        s["proj"].add(x)
    b = s["mesh"].mass(s["f"], s["b"])
    return {"b": b, "guess": s["proj"].project(b, s["z"])}


# ---------------------------------------------------------------------------
# what one pass cannot do without
def _points(case):
    return case["nx"] * case["ny"] * case["nz"] * (case["N"] + 1) ** 3


def _flops(N):
    """Of the local operator per point: six contractions and the 15 of the metric product."""
    return 12 * (N + 1) + 15


def work(case):
    kind = case["kind"]
    if kind == "batch":
        # one iteration of every system, times a modest count: each mesh's factors, diagonal and vectors
        n = sum(nel[0] * nel[1] * nel[2] * (N + 1) ** 3 for N, nel, _ in _boxes(case, 0))
        f = sum(nel[0] * nel[1] * nel[2] * (N + 1) ** 3 * _flops(N) for N, nel, _ in _boxes(case, 0))
        return {"bytes": 100 * 137.0 * n, "flops": 100.0 * f}
    n, N = _points(case), case["N"]
    if kind == "apply":
        # u, six factors (h1 and h2 B) in, w out
        return {"bytes": float(n * (10 if case["helm"] else 8) * (4 if case["dtype"] == "f32" else 8)),
                "flops": float(n * _flops(N))}
    if kind == "iterate":
        # per iteration: r, D^-1, p, x, w, multiplicity and six factors in; p, x, r, w out
        return {"bytes": 137.0 * n * case["iters"], "flops": float(n * (_flops(N) + 12) * case["iters"])}
    if kind == "solve":
        per = 137.0 if case["precision"] == "fp64" else 69.0
        return {"bytes": 200 * per * n, "flops": 200.0 * n * (_flops(N) + 12)}
    if kind == "precond":
        # r and the diagonal in, z out; with Schwarz the six contractions of (N+3)^4 per element
        e = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": 24.0 * n, "flops": float(12 * (N + 3) ** 4 * e if case["schwarz"] else 20 * n)}
    # each solution is read, applied and orthogonalised against those before it
    v = case["vectors"]
    return {"bytes": n * 8.0 * (v * (8 + 2) + 2 * v * (v - 1) + v + 4), "flops": float(n * v * (_flops(N) + 8 * v))}


# ---------------------------------------------------------------------------
# the mathematics in 64 bits, without the engine
def _gll(N):
    """GLL nodes, weights and the derivative matrix of the Lagrange basis."""
    c = np.zeros(N + 1)
    c[N] = 1.0
    L = np.polynomial.legendre
    d1 = L.legder(c)
    x = np.concatenate([[-1.0], np.sort(L.legroots(d1).real) if N > 1 else [], [1.0]])
    for _ in range(4):  # polish the roots of P_N'
        if N > 1:
            x[1:-1] -= L.legval(x[1:-1], d1) / L.legval(x[1:-1], L.legder(d1))
    x = 0.5 * (x - x[::-1])
    w = 2.0 / (N * (N + 1) * L.legval(x, c) ** 2)
    diff = x[:, None] - x[None, :] + np.eye(N + 1)
    lam = 1.0 / np.prod(diff, axis=1)
    D = lam[None, :] / lam[:, None] / diff
    np.fill_diagonal(D, 0.0)
    np.fill_diagonal(D, -D.sum(axis=1))
    return x, w, D


class _Ref:
    """A structured mesh and its operators in torch FP64.  Element vectors are
    [E, k, j, i]; homogeneous Dirichlet walls on every non-periodic face."""

    chunk_points = 6_000_000

    def __init__(self, case, seed):
        self.N, self.nel, self.per = case["N"], _nel(case), _periodic(case)
        self.pipe = case["map"] == "pipe"
        P = self.P = self.N + 1
        self.E = self.nel[0] * self.nel[1] * self.nel[2]
        xi, w, D = _gll(self.N)
        t = lambda a: torch.as_tensor(a, dtype=F64, device="cuda")  # noqa: E731
        self.xi, self.w, self.D = t(xi), t(w), t(D)
        self.verts = None if self.pipe else t(_vertices(self.nel, seed)).view(self.nel[2] + 1, self.nel[1] + 1,
                                                                             self.nel[0] + 1, 3)
        self.ext = [self.nel[d] * self.N + (0 if self.per[d] else 1) for d in range(3)]
        self.n_global = self.ext[0] * self.ext[1] * self.ext[2]
        self.step = max(1, self.chunk_points // P ** 3)
        self.h1 = self.h2 = None
        self._G = self._B = None

    def chunks(self):
        return [(a, min(self.E, a + self.step)) for a in range(0, self.E, self.step)]

    def position(self, a, b):
        e = torch.arange(a, b, device="cuda")
        nx, ny = self.nel[0], self.nel[1]
        return e % nx, (e // nx) % ny, e // (nx * ny)

    def lattice(self, a, b, lo=0, hi=None):
        """Per axis the lattice coordinates of GLL indices lo..hi of elements
        [a, b), wrapped on periodic axes, and whether they exist."""
        i = torch.arange(lo, (self.N if hi is None else hi) + 1, device="cuda")
        out = []
        for d, e in enumerate(self.position(a, b)):
            X = e[:, None] * self.N + i[None, :]
            if self.per[d]:
                X = X % self.ext[d]
            out.append((X, (X >= 0) & (X < self.ext[d])))
        return out

    def gid(self, a, b):
        (X, _), (Y, _), (Z, _) = self.lattice(a, b)
        return X[:, None, None, :] + self.ext[0] * (Y[:, None, :, None] + self.ext[1] * Z[:, :, None, None])

    def mask(self):
        """1 at interior nodes, 0 on the walls, per global node."""
        m = torch.ones(self.ext[2], self.ext[1], self.ext[0], dtype=F64, device="cuda")
        for d in range(3):
            if not self.per[d]:
                v = m.movedim(2 - d, 0)
                v[0] = 0.0
                v[-1] = 0.0
        return m.reshape(-1)

    def coords(self, a, b):
        f = 0.5 * (self.xi + 1.0)
        ex, ey, ez = self.position(a, b)
        if self.pipe:
            lo, hi = (-1.0, -1.0, 0.0), (1.0, 1.0, 10.0)
            c = [lo[d] + (e[:, None] + f[None, :]) * ((hi[d] - lo[d]) / self.nel[d]) for d, e in
                 enumerate((ex, ey, ez))]
            X, Y = c[0][:, None, None, :], c[1][:, None, :, None]
            shape = (b - a, self.P, self.P, self.P)
            return ((X * torch.sqrt(1 - 0.5 * Y * Y)).expand(shape), (Y * torch.sqrt(1 - 0.5 * X * X)).expand(shape),
                    c[2][:, :, None, None].expand(shape))
        F = torch.stack([1.0 - f, f])
        out = 0.0
        for c in range(8):
            cx, cy, cz = c & 1, (c >> 1) & 1, c >> 2
            wgt = F[cz][:, None, None] * F[cy][None, :, None] * F[cx][None, None, :]
            out = out + wgt[None, ..., None] * self.verts[ez + cz, ey + cy, ex + cx][:, None, None, None, :]
        return out[..., 0], out[..., 1], out[..., 2]

    def global_coords(self):
        out = [torch.empty(self.n_global, dtype=F64, device="cuda") for _ in range(3)]
        for a, b in self.chunks():
            g = self.gid(a, b).reshape(-1)
            for o, c in zip(out, self.coords(a, b)):
                o[g] = c.reshape(-1)
        return out

    def grad(self, u):
        """The three reference derivatives of element vectors."""
        P, n = self.P, u.shape[0]
        r = (u.reshape(-1, P) @ self.D.T).view(u.shape)
        s = torch.matmul(self.D, u.reshape(-1, P, P)).view(u.shape)
        t = torch.matmul(self.D, u.reshape(n, P, P * P)).view(u.shape)
        return r, s, t

    def grad_t(self, r, s, t):
        P, n = self.P, r.shape[0]
        DT = self.D.T.contiguous()
        out = (r.reshape(-1, P) @ self.D).view(r.shape)
        out = out + torch.matmul(DT, s.reshape(-1, P, P)).view(r.shape)
        return out + torch.matmul(DT, t.reshape(n, P, P * P)).view(r.shape)

    def factors(self, a, b):
        """The six metric factors and the mass of elements [a, b)."""
        J = [self.grad(c.contiguous()) for c in self.coords(a, b)]  # J[x][r]
        C = [[J[(x + 1) % 3][(r + 1) % 3] * J[(x + 2) % 3][(r + 2) % 3]
              - J[(x + 1) % 3][(r + 2) % 3] * J[(x + 2) % 3][(r + 1) % 3] for r in range(3)] for x in range(3)]
        det = sum(J[0][r] * C[0][r] for r in range(3))
        W = self.w[:, None, None] * self.w[None, :, None] * self.w[None, None, :]
        G = [W * sum(C[x][p] * C[x][q] for x in range(3)) / det for p, q in
             ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))]
        B = W * det
        if self.pipe:
            # the map is singular at the square's corners: those points are dropped
            ex, ey, _ = self.position(a, b)
            N = self.N
            for i, x in ((0, 0), (N, self.nel[0] - 1)):
                for j, y in ((0, 0), (N, self.nel[1] - 1)):
                    at = ((ex == x) & (ey == y)).nonzero().view(-1)
                    for v in G + [B]:
                        v[at, :, j, i] = 0.0
        return G, B

    def keep_factors(self):
        self._G = [self.factors(a, b) for a, b in self.chunks()]
        self._ids = [self.gid(a, b) for a, b in self.chunks()]
        return self

    def _parts(self):
        for q, (a, b) in enumerate(self.chunks()):
            G, B = self._G[q] if self._G else self.factors(a, b)
            yield a, b, G, B, (self._ids[q] if self._G else self.gid(a, b))

    def local(self, u, G, B, a, b):
        r, s, t = self.grad(u)
        g = [G[0] * r + G[3] * s + G[4] * t, G[3] * r + G[1] * s + G[5] * t, G[4] * r + G[5] * s + G[2] * t]
        if self.h1 is not None:
            h = self.h1.view(self.E, self.P, self.P, self.P)[a:b]
            g = [h * v for v in g]
        w = self.grad_t(*g)
        if self.h2 is not None:
            w = w + self.h2.view(self.E, self.P, self.P, self.P)[a:b] * B * u
        return w

    def apply(self, vg):
        """mask(Q^T A_L Q v) on global vectors."""
        out = torch.zeros(self.n_global, dtype=F64, device="cuda")
        for a, b, G, B, g in self._parts():
            out.index_add_(0, g.reshape(-1), self.local(vg[g], G, B, a, b).reshape(-1))
        return out * self.mask()

    def spread(self, vg):
        """Global values at every local node."""
        return torch.cat([vg[self.gid(a, b)].reshape(-1) for a, b in self.chunks()])

    def assemble(self, make):
        """Sum over the copies of make(a, b, G, B)."""
        out = torch.zeros(self.n_global, dtype=F64, device="cuda")
        for a, b, G, B, g in self._parts():
            out.index_add_(0, g.reshape(-1), make(a, b, G, B).reshape(-1))
        return out

    def diagonal(self):
        D2, d = self.D ** 2, torch.diagonal(self.D)

        def make(a, b, G, B):
            P, n = self.P, b - a
            D2T = D2.T.contiguous()
            v = (G[0].reshape(-1, P) @ D2).view(G[0].shape)
            v = v + torch.matmul(D2T, G[1].reshape(-1, P, P)).view(G[0].shape)
            v = v + torch.matmul(D2T, G[2].reshape(n, P, P * P)).view(G[0].shape)
            di, dj, dk = d[None, None, :], d[None, :, None], d[:, None, None]
            return v + 2 * (di * dj * G[3] + di * dk * G[4] + dj * dk * G[5])

        return self.assemble(make)

    def pcg(self, b, iters=None, tol=1e-13, limit=20000):
        """Jacobi-PCG on global vectors: `iters` steps, or to `tol`."""
        mask = self.mask()
        inv = torch.where(mask > 0, 1.0 / self.diagonal(), torch.zeros_like(mask))
        x, r = torch.zeros_like(b), b.clone()
        z = inv * r
        p, rho = z.clone(), torch.dot(r, z)
        stop = tol * float(b.norm())
        for it in range(limit if iters is None else iters):
            w = self.apply(p)
            alpha = rho / torch.dot(p, w)
            x += alpha * p
            r -= alpha * w
            if iters is None and it % 8 == 7 and float(r.norm()) <= stop:
                break
            z = inv * r
            new = torch.dot(r, z)
            p = z + (new / rho) * p
            rho = new
        return x

    # -- the preconditioner of Eq. 6 -----------------------------------------
    def coarse(self, r, steps, fraction=0.05):
        """P C(A0) P^T r: trilinear vertex hats, the Galerkin operator, and
        Chebyshev steps on [fraction b, b] with b its largest row sum."""
        P, mask = self.P, self.mask()
        q = torch.stack([0.5 * (1 - self.xi), 0.5 * (1 + self.xi)])
        hats = torch.stack([q[c >> 2][:, None, None] * q[(c >> 1) & 1][None, :, None] * q[c & 1][None, None, :]
                            for c in range(8)])
        vd = [self.nel[d] + 1 - self.per[d] for d in range(3)]
        nv = vd[0] * vd[1] * vd[2]
        mult = self.assemble(lambda a, b, G, B: torch.ones(b - a, P, P, P, dtype=F64, device="cuda"))
        verts, r0, blocks = [], torch.zeros(nv, dtype=F64, device="cuda"), []
        for a, b, G, B, g in self._parts():
            ex, ey, ez = self.position(a, b)
            v = torch.stack([(ex + (c & 1)) % vd[0] + vd[0] * ((ey + ((c >> 1) & 1)) % vd[1] + vd[1] * (
                (ez + (c >> 2)) % vd[2])) for c in range(8)], dim=1)
            verts.append(v)
            live = mask[g]
            f = (live * r[g] / mult[g]).reshape(b - a, -1)
            r0.index_add_(0, v.reshape(-1), (f @ hats.reshape(8, -1).T).reshape(-1))
            cols = [self.local(live * hats[c], G, B, a, b) * live for c in range(8)]
            blocks.append(torch.stack([w.reshape(b - a, -1) @ hats.reshape(8, -1).T for w in cols], dim=2))
        v, K = torch.cat(verts), torch.cat(blocks)  # K[e, row, col]
        at = torch.stack([v[:, :, None].expand(-1, 8, 8).reshape(-1), v[:, None, :].expand(-1, 8, 8).reshape(-1)])
        A0 = torch.sparse_coo_tensor(at, K.reshape(-1), (nv, nv)).coalesce()
        i, val = A0.indices(), A0.values()
        diag = torch.zeros(nv, dtype=F64, device="cuda")
        diag[i[0][i[0] == i[1]]] = val[i[0] == i[1]]
        inv = torch.where(diag > 0, 1.0 / diag, torch.zeros_like(diag))
        hi = float((torch.zeros_like(diag).index_add_(0, i[0], val.abs()) * inv).max())
        theta, delta = 0.5 * hi * (1 + fraction), 0.5 * hi * (1 - fraction)
        sigma, z, res = theta / delta, torch.zeros_like(r0), r0 * (diag > 0)
        rho, d = 1.0 / sigma, r0 * inv / theta
        for _ in range(steps):
            z = z + d
            res = res - torch.zeros_like(res).index_add_(0, i[0], val * d[i[1]])
            new = 1.0 / (2.0 * sigma - rho)
            d = new * rho * d + (2.0 * new / delta) * inv * res
            rho = new
        out = torch.zeros(self.n_global, dtype=F64, device="cuda")
        for (a, b), vv in zip(self.chunks(), verts):
            out[self.gid(a, b).reshape(-1)] = (z[vv] @ hats.reshape(8, -1)).reshape(-1)
        return out * mask

    def _modes(self, left, right):
        """Generalised eigenvectors and values of the 1-D extended element of
        length 2 with the given sides (0 a neighbour, 1 a wall), in the
        extended index range -1..N+1; absent indices give zero rows."""
        N, n = self.N, self.N + 3
        D, w = self.D.cpu().numpy(), self.w.cpu().numpy()
        Ke, K, B = D.T @ np.diag(w) @ D, np.zeros((3 * N + 1, 3 * N + 1)), np.zeros(3 * N + 1)
        for p in [1] + ([0] if left == 0 else []) + ([2] if right == 0 else []):
            K[p * N:p * N + N + 1, p * N:p * N + N + 1] += Ke
            B[p * N:p * N + N + 1] += w
        keep = np.arange(-1 if left == 0 else 1, (N + 1 if right == 0 else N - 1) + 1)
        s = 1.0 / np.sqrt(B[N + keep])
        lam, Q = np.linalg.eigh(K[np.ix_(N + keep, N + keep)] * s[:, None] * s[None, :])
        S, L = np.zeros((n, n)), np.full(n, np.inf)
        S[keep + 1, :len(keep)] = s[:, None] * Q
        L[:len(keep)] = lam
        return S, L

    def schwarz(self, r):
        """Sum over the elements extended by one node layer of their separable
        local solves (mean edge lengths)."""
        out = torch.zeros(self.n_global, dtype=F64, device="cuda")
        tables = {}
        for l in (0, 1):
            for rr in (0, 1):
                tables[l, rr] = [torch.as_tensor(v, device="cuda") for v in self._modes(l, rr)]
        N = self.N
        for a, b in self.chunks():
            xyz = torch.stack(self.coords(a, b), dim=-1)[:, ::N, ::N, ::N]  # the corners [e, k, j, i, :]
            S, lam = [], []
            for d, e in enumerate(self.position(a, b)):
                c = xyz.movedim(3 - d, 1)
                ell = (c[:, 1] - c[:, 0]).norm(dim=-1).mean(dim=(1, 2))
                wall = [(e == 0) & (not self.per[d]), (e == self.nel[d] - 1) & (not self.per[d])]
                Sd = torch.zeros(b - a, N + 3, N + 3, dtype=F64, device="cuda")
                Ld = torch.zeros(b - a, N + 3, dtype=F64, device="cuda")
                for (l, rr), (St, Lt) in tables.items():
                    at = ((wall[0] == bool(l)) & (wall[1] == bool(rr))).nonzero().view(-1)
                    Sd[at] = St * torch.sqrt(2.0 / ell[at])[:, None, None]
                    Ld[at] = Lt * (4.0 / ell[at] ** 2)[:, None]
                S.append(Sd)
                lam.append(Ld)
            (X, okx), (Y, oky), (Z, okz) = self.lattice(a, b, -1, N + 1)
            ok = okx[:, None, None, :] & oky[:, None, :, None] & okz[:, :, None, None]
            g = X[:, None, None, :] + self.ext[0] * (Y[:, None, :, None] + self.ext[1] * Z[:, :, None, None])
            g = torch.where(ok, g, torch.zeros_like(g))
            u = torch.where(ok, r[g], torch.zeros((), dtype=F64, device="cuda"))
            n = N + 3

            def turn(u, M):
                # along r, s and t: u <- M_d u
                u = torch.matmul(u.reshape(b - a, n * n, n), M[0].transpose(1, 2).contiguous()).view(-1, n, n, n)
                u = torch.matmul(M[1][:, None], u)
                return torch.matmul(M[2], u.reshape(b - a, n, n * n)).view(-1, n, n, n)

            y = turn(u, [m.transpose(1, 2).contiguous() for m in S])
            y = y / (lam[0][:, None, None, :] + lam[1][:, None, :, None] + lam[2][:, :, None, None])
            z = turn(y, S)
            out.index_add_(0, g.reshape(-1), torch.where(ok, z, torch.zeros_like(z)).reshape(-1))
        return out * self.mask()


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for N, nel, vs in _boxes(case, seed):
            ref = _Ref(_box_case(N, nel), vs).keep_factors()
            out.append(ref.spread(ref.pcg(_rhs_values(ref.n_global, vs) * ref.mask())))
        return out
    ref = _Ref(case, seed)
    n_local = _points(case)
    if kind == "apply":
        if case["helm"]:
            ref.h1, ref.h2 = _random(n_local, seed + 1, 0.5, 2.0), _random(n_local, seed + 2, 0.0, 3.0)
        u = _random(ref.n_global, seed) * ref.mask()
        if case["dtype"] == "f32":
            u = u.float().double()
        return ref.spread(ref.apply(u))
    if kind == "projection":
        ref.keep_factors()
        f = _random(n_local, seed).view(ref.E, ref.P, ref.P, ref.P)
        b = ref.assemble(lambda p, q, G, B: B * f[p:q]) * ref.mask()
        X = torch.stack([v * ref.mask() for v in _smooth_values(ref, seed, case["vectors"])])
        AX = torch.stack([ref.apply(x) for x in X])
        gram = X @ AX.T
        coef = torch.linalg.solve(0.5 * (gram + gram.T), X @ b)
        return {"b": ref.spread(b), "guess": ref.spread(coef @ X)}
    b = _rhs_values(ref.n_global, seed) * ref.mask()
    if kind == "precond":
        z = ref.coarse(b, case["coarse"])
        if case["schwarz"]:
            return ref.spread(z + ref.schwarz(b))
        mask = ref.mask()
        return ref.spread(z + torch.where(mask > 0, b / ref.diagonal(), torch.zeros_like(b)))
    ref.keep_factors()
    return ref.spread(ref.pcg(b, case["iters"] if kind == "iterate" else None))
