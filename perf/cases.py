"""Performance cases: the work that a flow solver hands to this library.

Every case is one pass through the public Python entry points on a deformed
box of hexahedra (the mesh family of the tests and of bench.py): operator
applications, right-hand sides already assembled, and whole solves.  A mesh,
its order and everything the library keeps for it (numbering, factors,
preconditioner) are set up once and serve every later right-hand side, as in
a time-stepping program; the vectors are new for every seed.

The reference values are computed here with plain torch in 64 bits on the
node lattice of the box: the operator applied by dense 1D contractions, and
for the solves the field that the right-hand side was made from.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2207_07098_amd as sem

TWO_PI = 2.0 * math.pi


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------
def _case(kind, K, N, precision="fp64", **more):
    kx, ky, kz = (K, K, K) if isinstance(K, int) else K
    return dict(kind=kind, kx=kx, ky=ky, kz=kz, N=N, precision=precision, **more)


def listed():
    def named(name, c):
        c["name"] = name
        return c
    return [
        # one operator application on the smallest mesh of the tests: what
        # counts is the latency of the call
        named("ax_4_N5", _case("ax", 4, 5)),
        # the assembled E-vector form Q Q^T A_L u_L, the form in which codes
        # with element-local storage use the operator, at an ordinary size
        named("evec_24_N7", _case("evec", 24, 7)),
        # Jacobi-PCG on the smallest mesh: launches and host round trips
        named("cg_4_N5", _case("cg", 4, 5)),
        # velocity solve h1 A + h2 B of a time step at an ordinary size
        named("helmholtz_24_N7", _case("helmholtz", 24, 7)),
        # pressure solves of five successive time steps, each projected on
        # the earlier ones, on a mesh with different element counts per axis
        # and an even order
        named("projection_13x11x9_N8", _case("projection", (13, 11, 9), 8, steps=5)),
        # pressure solver (GMRES, overlapping Schwarz, coarse grid) on a
        # small mesh: latency of each iteration's chain
        named("gmres_8_N7", _case("gmres", 8, 7)),
        # the same in mixed precision on a ragged mesh at an even order
        named("gmres_21x18x16_N6_fp32", _case("gmres", (21, 18, 16), 6, "fp32")),
        # 32 independent problems of different sizes and orders in one batch
        named("batch_32", dict(kind="batch", problems=32, kmin=2, kmax=12, mesh_seed=7,
                               precision="fp64")),
        # the largest mesh: one operator application in FP64 and with 16-bit
        # factors, the mixed-precision solve, and the FP64 pressure solve
        named("ax_48_N7", _case("ax", 48, 7)),
        named("ax_48_N7_fp16", _case("ax", 48, 7, "fp16")),
        named("cg_48_N7_fp32", _case("cg", 48, 7, "fp32")),
        named("gmres_48_N7", _case("gmres", 48, 7)),
    ]


def draw(rng):
    kind = rng.choice(["ax", "ax", "evec", "cg", "helmholtz", "projection", "gmres", "gmres",
                       "batch"])
    if kind == "batch":
        return dict(kind="batch", problems=rng.randint(3, 32), kmin=2, kmax=rng.randint(4, 12),
                    mesh_seed=rng.randint(0, 10 ** 6), precision="fp64")
    # unique nodes spread over the logarithm of the range, split unevenly
    # over the axes; whole solves stay at meshes that they finish quickly
    top = {"ax": 3.8e7, "evec": 1.2e7, "cg": 6e6, "helmholtz": 1.2e7, "projection": 2e6,
           "gmres": 1.2e7}[kind]
    N = rng.choice([3, 4, 5, 6, 7, 7, 7, 8, 9, 10] + ([2, 11, 13] if kind in ("ax", "evec") else []))
    nodes = math.exp(rng.uniform(math.log(5e3), math.log(0.8 * top)))
    side = max(3.0, (nodes ** (1.0 / 3.0) - 1.0) / N)
    ks = [max(3, int(round(side * math.exp(rng.uniform(-0.25, 0.25))))) for _ in range(3)]
    while np.prod([k * N + 1 for k in ks]) > top:
        ks[int(np.argmax(ks))] -= 1
    precision = {"ax": ["fp64", "fp64", "fp32", "fp16", "bf16"], "evec": ["fp64", "fp32"],
                 "cg": ["fp64", "fp32", "fp16"], "helmholtz": ["fp64"], "projection": ["fp64"],
                 "gmres": ["fp64", "fp32"]}[kind]
    c = _case(kind, tuple(ks), N, rng.choice(precision))
    if kind == "projection":
        c["steps"] = rng.randint(2, 6)
    return c


# ---------------------------------------------------------------------------
# the box: lattice numbering, GLL rule and geometry in plain torch
# ---------------------------------------------------------------------------
def gll_rule(N):
    """GLL nodes, weights and derivative matrix in 64 bits."""
    L = np.polynomial.legendre.Legendre.basis(N)
    dL, ddL = L.deriv(), L.deriv(2)
    x = np.sort(np.real(dL.roots())) if N > 1 else np.zeros(0)
    for _ in range(3):
        x = x - dL(x) / ddL(x) if N > 1 else x
    x = np.concatenate([[-1.0], x, [1.0]])
    x = 0.5 * (x - x[::-1])
    rho = 2.0 / (N * (N + 1) * L(x) ** 2)
    D = np.zeros((N + 1, N + 1))
    for i in range(N + 1):
        for j in range(N + 1):
            if i != j:
                D[i, j] = L(x[i]) / (L(x[j]) * (x[i] - x[j]))
    D[0, 0], D[N, N] = -N * (N + 1) / 4.0, N * (N + 1) / 4.0
    return x, rho, D


class Box:
    """[0, 2 pi]^3 with kx*ky*kz elements of order N, every node moved by
    0.05 h sin x sin y sin z (h the smallest element width; zero on the faces),
    Dirichlet conditions on all faces."""

    def __init__(self, kx, ky, kz, N):
        self.K, self.N = (kx, ky, kz), N
        self.num_elements = kx * ky * kz
        self.num_vertices = (kx + 1) * (ky + 1) * (kz + 1)
        e = np.arange(self.num_elements, dtype=np.int64)
        pos = (e % kx, (e // kx) % ky, e // (kx * ky))
        self.corner_ids = np.stack(
            [pos[0] + (c & 1) + (kx + 1) * (pos[1] + ((c >> 1) & 1)
                                            + (ky + 1) * (pos[2] + (c >> 2))) for c in range(8)],
            axis=1)
        self.face_bc = np.stack([pos[d // 2] == (0 if d % 2 == 0 else self.K[d // 2] - 1)
                                 for d in range(6)], axis=1).astype(np.uint8)
        self.x1, self.rho, self.D = gll_rule(N)

    def axis(self, d, dev):
        """Undeformed coordinates of the lattice nodes along one axis."""
        k, N = self.K[d], self.N
        n = torch.arange(k * N + 1, device=dev)
        e = torch.clamp(n // N, max=k - 1)
        xi = torch.from_numpy(self.x1).to(dev)[n - e * N]
        return (e + 0.5 * (xi + 1.0)) * (TWO_PI / k)

    def lattice(self, dev):
        """Coordinates of all lattice nodes, each [nz, ny, nx]."""
        x, y, z = self.axis(0, dev), self.axis(1, dev), self.axis(2, dev)
        s = (torch.sin(z)[:, None, None] * torch.sin(y)[None, :, None]
             * torch.sin(x)[None, None, :]) * (0.05 * TWO_PI / max(self.K))
        return x[None, None, :] + s, y[None, :, None] + s, z[:, None, None] + s

    def element_nodes(self, dev):
        """Lattice index of every local point, [E, n1, n1, n1] (i fastest)."""
        kx, ky, kz = self.K
        N = self.N
        e = torch.arange(self.num_elements, device=dev)
        o = torch.arange(N + 1, device=dev)
        I = ((e % kx) * N)[:, None] + o
        J = (((e // kx) % ky) * N)[:, None] + o
        L = ((e // (kx * ky)) * N)[:, None] + o
        return (I[:, None, None, :] + (kx * N + 1) * (J[:, None, :, None]
                + (ky * N + 1) * L[:, :, None, None]))

    def solver_lattice(self, dev):
        """Lattice index of every unique node in the library's vector order:
        nodes on element boundaries by first appearance (element, then local
        point), then element interiors."""
        N, n1 = self.N, self.N + 1
        own = []
        for d in range(3):
            n = torch.arange(self.K[d] * N + 1, device=dev)
            e = torch.clamp((n + N - 1) // N - 1, min=0)
            own.append((e, n - e * N))
        (ex, i), (ey, j), (ez, k) = own
        e = ex[None, None, :] + self.K[0] * (ey[None, :, None] + self.K[1] * ez[:, None, None])
        l = i[None, None, :] + n1 * (j[None, :, None] + n1 * k[:, None, None])
        edge = [((v == 0) | (v == N)) for v in (i, j, k)]
        inner = ~(edge[0][None, None, :] | edge[1][None, :, None] | edge[2][:, None, None])
        key = e * n1 ** 3 + l + inner * (self.num_elements * n1 ** 3)
        return torch.argsort(key.reshape(-1))

    def mask(self, dev):
        m = torch.ones([k * self.N + 1 for k in reversed(self.K)], dtype=torch.float64, device=dev)
        m[0], m[-1], m[:, 0], m[:, -1], m[:, :, 0], m[:, :, -1] = 0, 0, 0, 0, 0, 0
        return m.reshape(-1)


class Reference:
    """The operator of a box in plain torch, 64 bits."""

    def __init__(self, box, dev):
        self.box, self.dev = box, dev
        self.nodes = box.element_nodes(dev).reshape(-1)
        self.shape = (box.num_elements,) + (box.N + 1,) * 3
        self.D = torch.from_numpy(box.D).to(dev)
        self.mask = box.mask(dev)
        self.n = self.mask.numel()
        self.order = box.solver_lattice(dev)
        self.G = self.B = None

    def grad(self, v):
        D, Dt = self.D, self.D.t().contiguous()
        n = self.shape[1]
        r = (v.reshape(-1, n) @ Dt).reshape(self.shape)
        s = (v.transpose(2, 3).reshape(-1, n) @ Dt).reshape(self.shape).transpose(2, 3)
        t = (v.reshape(-1, n, n * n).transpose(1, 2).reshape(-1, n) @ Dt)
        t = t.reshape(-1, n * n, n).transpose(1, 2).reshape(self.shape)
        return r, s, t

    def grad_t(self, r, s, t):
        D = self.D.contiguous()
        n = self.shape[1]
        w = (r.reshape(-1, n) @ D).reshape(self.shape)
        w = w + (s.transpose(2, 3).reshape(-1, n) @ D).reshape(self.shape).transpose(2, 3)
        q = t.reshape(-1, n, n * n).transpose(1, 2).reshape(-1, n) @ D
        return w + q.reshape(-1, n * n, n).transpose(1, 2).reshape(self.shape)

    def coordinates(self):
        return [c.expand(self.order_shape()).reshape(-1)[self.nodes].reshape(self.shape)
                for c in self.box.lattice(self.dev)]

    def order_shape(self):
        return [k * self.box.N + 1 for k in reversed(self.box.K)]

    def geometry(self):
        """Factors (11, 22, 33, 12, 13, 23) and lumped mass."""
        if self.G is not None:
            return
        J = [self.grad(c) for c in self.coordinates()]          # J[l][s] = dx_l / dr_s
        A = []
        for s in range(3):
            a, b = (s + 1) % 3, (s + 2) % 3
            A.append([J[(l + 1) % 3][a] * J[(l + 2) % 3][b] - J[(l + 2) % 3][a] * J[(l + 1) % 3][b]
                      for l in range(3)])
        det = sum(J[l][0] * A[0][l] for l in range(3))
        rho = torch.from_numpy(self.box.rho).to(self.dev)
        w = rho[:, None, None] * rho[None, :, None] * rho[None, None, :]
        f = w / det
        self.G = [f * sum(A[p][l] * A[q][l] for l in range(3))
                  for p, q in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))]
        self.B = w * det

    def local(self, v):
        """A_L on an E-vector."""
        self.geometry()
        g = self.G
        r, s, t = self.grad(v)
        return self.grad_t(g[0] * r + g[3] * s + g[4] * t, g[3] * r + g[1] * s + g[5] * t,
                           g[4] * r + g[5] * s + g[2] * t)

    def gather(self, lat):
        return lat[self.nodes].reshape(self.shape)

    def scatter(self, w):
        y = torch.zeros(self.n, dtype=torch.float64, device=self.dev)
        return y.index_add_(0, self.nodes, w.reshape(-1)) * self.mask

    def apply(self, lat, h1=1.0, h2=0.0):
        """M Q^T (h1 A_L + h2 B_L) Q M on a lattice vector."""
        v = self.gather(lat * self.mask)
        w = self.local(v)
        if h2:
            w = h1 * w + h2 * self.B * v
        return self.scatter(w)

    def to_solver(self, lat):
        return lat[self.order]

    def from_solver(self, u):
        lat = torch.empty_like(u)
        lat[self.order] = u
        return lat


# ---------------------------------------------------------------------------
# what a program keeps between time steps: the last mesh and its operator
# ---------------------------------------------------------------------------
class Kept:
    def __init__(self, kx, ky, kz, N, precisions):
        dev = torch.device("cuda")
        self.box = Box(kx, ky, kz, N)
        self.ref = Reference(self.box, dev)
        xyz = torch.stack(self.ref.coordinates(), dim=1).cpu().numpy()
        self.op = sem.Operator(self.box, N, precisions=precisions, gll_xyz=xyz)
        self.pressure = self.projection = None


_kept = {}
H1, H2 = 0.01, 20.0            # velocity operator of bench.py


def _keep(c):
    """The operator of the case's mesh; only the last mesh is kept."""
    key = (c["kx"], c["ky"], c["kz"], c["N"], c["kind"] == "helmholtz")
    low = {"fp64": "fp32"}.get(c["precision"], c["precision"])
    k = _kept.get(key)
    if k is None or low not in k.op.precisions:
        _kept.clear()
        # the 48^3 cases share one operator, which then holds both copies
        prec = ("fp64", "fp32", "fp16") if low in ("fp32", "fp16") else ("fp64", low)
        k = Kept(c["kx"], c["ky"], c["kz"], c["N"], prec)
        if c["kind"] == "helmholtz":
            k.op.set_helmholtz(H1, H2)
        _kept[key] = k
    return k


def _field(box, seed, dev, step=0):
    """A smooth field on the lattice that vanishes on the boundary: sine modes
    of several scales with random amplitudes (and, for a sequence, a source
    that moves with the step)."""
    rng = np.random.default_rng([seed, 11])
    x, y, z = box.axis(0, dev), box.axis(1, dev), box.axis(2, dev)
    out = 0.0
    for m in range(6):
        k = rng.integers(1, 7, 3) * 0.5
        a = rng.uniform(0.5, 1.0) * rng.choice([-1.0, 1.0]) / (1.0 + 0.3 * float(k.sum()))
        out = out + a * (torch.sin(k[2] * z)[:, None, None] * torch.sin(k[1] * y)[None, :, None]
                         * torch.sin(k[0] * x)[None, None, :])
    if step:
        c = rng.uniform(2.0, 4.0, 3)
        v = rng.uniform(-0.15, 0.15, 3)
        g = [torch.sin(0.5 * q) * torch.exp(-(q - (c[d] + v[d] * step)) ** 2)
             for d, q in enumerate((x, y, z))]
        out = out + 2.0 * g[2][:, None, None] * g[1][None, :, None] * g[0][None, None, :]
    return out.reshape(-1)


def _batch_meshes(c):
    rng = np.random.default_rng(c["mesh_seed"])
    return [dict(kind="cg", kx=int(k[0]), ky=int(k[1]), kz=int(k[2]), N=int(n), precision="fp64")
            for k, n in ((rng.integers(c["kmin"], c["kmax"] + 1, 3), rng.choice([5, 7, 9]))
                         for _ in range(c["problems"]))]


def _vector(c, seed, dev):
    """The vector an operator application acts on, with its type."""
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    n = int(np.prod([k * c["N"] + 1 for k in (c["kx"], c["ky"], c["kz"])]))
    if c["kind"] == "evec":
        n = c["kx"] * c["ky"] * c["kz"] * (c["N"] + 1) ** 3
    u = torch.rand(n, generator=g, dtype=torch.float64, device=dev) * 2.0 - 1.0
    return u if c["precision"] == "fp64" else u.float()


def prepare(case, seed):
    c, dev = case, torch.device("cuda")
    kind = c["kind"]
    if kind == "batch":
        key = ("batch", c["problems"], c["kmin"], c["kmax"], c["mesh_seed"])
        if key not in _kept:
            _kept.clear()
            parts = [Kept(m["kx"], m["ky"], m["kz"], m["N"], ("fp64", "fp32"))
                     for m in _batch_meshes(c)]
            _kept[key] = (parts, sem.Batch([p.op for p in parts]))
        parts, batch = _kept[key]
        rhs = [p.ref.to_solver(p.ref.apply(_field(p.box, seed + 1000 * q, dev)))
               for q, p in enumerate(parts)]
        return dict(case=c, batch=batch, rhs=rhs)
    k = _keep(c)
    s = dict(case=c, op=k.op)
    if kind in ("ax", "evec"):
        s["u"] = _vector(c, seed, dev)
        s["y"] = torch.zeros_like(s["u"])
        return s
    h = (H1, H2) if kind == "helmholtz" else (1.0, 0.0)
    if kind == "projection":
        s["b"] = [k.ref.to_solver(k.ref.apply(_field(k.box, seed, dev, 1 + t)))
                  for t in range(c["steps"])]
        if k.projection is None:
            k.projection = sem.Projection(k.op)
        s["projection"] = k.projection
        return s
    s["b"] = k.ref.to_solver(k.ref.apply(_field(k.box, seed, dev), *h))
    k.ref.G = k.ref.B = None
    if kind == "gmres":
        if k.pressure is None:
            k.pressure = sem.PressureSolver(k.op)
        s["pressure"] = k.pressure
    return s


def run(state):
    c = state["case"]
    kind, prec = c["kind"], c["precision"]
    if kind == "ax":
        return state["op"].ax(state["u"], state["y"], precision=prec)
    if kind == "evec":
        return state["op"].ax_evec(state["u"], state["y"], precision=prec)
    if kind in ("cg", "helmholtz"):
        return state["op"].solve(state["b"], tol=1e-10, precision=prec)[0]
    if kind == "gmres":
        return state["pressure"].solve(state["b"], tol=1e-10, precision=prec)[0]
    if kind == "projection":
        p = state["projection"]
        p.reset()
        return [p.solve(b, tol=1e-10)[0] for b in state["b"]]
    return state["batch"].solve(state["rhs"], tol=1e-10)[0]


def exact(case, seed):
    c, dev = case, torch.device("cuda")
    kind = c["kind"]

    def solution(m, sd, step=0):
        box = Box(m["kx"], m["ky"], m["kz"], m["N"])
        return _field(box, sd, dev, step)[box.solver_lattice(dev)]

    if kind == "batch":
        return [solution(m, seed + 1000 * q) for q, m in enumerate(_batch_meshes(c))]
    if kind == "projection":
        return [solution(c, seed, 1 + t) for t in range(c["steps"])]
    if kind in ("cg", "helmholtz", "gmres"):
        return solution(c, seed)
    ref = Reference(Box(c["kx"], c["ky"], c["kz"], c["N"]), dev)
    u = _vector(c, seed, dev).double()
    if kind == "ax":
        return ref.to_solver(ref.apply(ref.from_solver(u)))
    return ref.gather(ref.scatter(ref.local(u.reshape(ref.shape)))).reshape(-1)


# ---------------------------------------------------------------------------
# work that a pass cannot do without
# ---------------------------------------------------------------------------
def _sizes(c):
    E, n1 = c["kx"] * c["ky"] * c["kz"], c["N"] + 1
    nl = E * n1 ** 3
    nu = int(np.prod([k * c["N"] + 1 for k in (c["kx"], c["ky"], c["kz"])]))
    return E, n1, nl, nu


def _operator(c, s, v):
    """Factors of s bytes and a map entry per local point, vectors of v bytes."""
    E, n1, nl, nu = _sizes(c)
    return nl * (6 * s + 4) + 2 * v * nu, (12 * n1 + 15) * nl


def _pcg_iterations(c):
    return 6.3 * c["N"] * max(c["kx"], c["ky"], c["kz"])


def _pcg(c, iterations, v):
    """Jacobi-PCG: the operator and ten more vector passes per iteration."""
    b, f = _operator(c, v, v)
    nu = _sizes(c)[3]
    return iterations * (b + 10 * v * nu), iterations * (f + 14 * nu)


def work(case):
    c = case
    kind = c["kind"]
    s = {"fp64": 8, "fp32": 4, "fp16": 2, "bf16": 2}[c["precision"]]
    v = 8 if c["precision"] == "fp64" else 4
    if kind == "batch":
        parts = [_pcg(m, _pcg_iterations(m), 8) for m in _batch_meshes(c)]
        b, f = (sum(q) for q in zip(*parts))
    elif kind == "ax":
        b, f = _operator(c, s, v)
    elif kind == "evec":
        E, n1, nl, nu = _sizes(c)
        b, f = nl * (6 * s + 2 * v) + 4 * E * (n1 ** 3 - (n1 - 2) ** 3), (12 * n1 + 15) * nl
    elif kind == "cg":
        b, f = _pcg(c, _pcg_iterations(c), v)
    elif kind == "helmholtz":
        E, n1, nl, nu = _sizes(c)
        b, f = _pcg(c, 37, 8)
        b += 37 * 8 * nl
    elif kind == "projection":
        b, f = _pcg(c, 0.8 * c["steps"] * _pcg_iterations(c), 8)
    else:
        # GMRES: per step one operator, the local solves (r, z, the
        # eigenvectors and maps once, six contractions of the extended box),
        # the coarse grid and two sweeps over half the basis on average
        E, n1, nl, nu = _sizes(c)
        steps, ne = 24, n1 + 2
        ob, of = _operator(c, v, v)
        fb = 2 * v * nu + E * (3 * ne * ne * v + 4 * ne ** 3)
        b = steps * (ob + fb + (steps + 6) * v * nu)
        f = steps * (of + E * 12 * ne ** 4 + 2 * steps * 2 * nu)
    return {"bytes": float(b), "flops": float(f)}
