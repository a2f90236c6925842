"""The work that programs built on libsem have it do, as cases that can be timed.

A case is a dict of plain values: the operation, the mesh recipe, the order and
the options of the call.  `prepare` makes what a program holds before the call
(the mesh handle, which it keeps over many calls, and new input vectors from a
seed), `run` is one pass through the public entry points, `work` counts what
the pass cannot do without, and `exact` gives its outputs from plain torch in
64 bits.

Meshes: "cube" is the unit cube with straight-edged elements whose interior
vertices are displaced at random by up to 5 % of the element size, Dirichlet
walls; "slab" is a [0,4]x[0,4]x[0,1] convection box, periodic in x and y,
Dirichlet plates, element layers clustered to the plates (tallest/lowest
height 20) and curved elements; "layers" is the unit cube with the same
clustering, curved elements and no Dirichlet node (constant null space).
"""

import math
from functools import lru_cache

import numpy as np
import torch

import paper_2501_13240_amd as sem
from paper_2501_13240_amd.autograd import sem_solve

DEV = "cuda"


def listed():
    return [
        # the operator on the smallest mesh in use: launch and call latency
        dict(name="ax_cube4_n7", op="ax", mesh="cube", nx=4, ny=4, nz=4, N=7, dtype="fp64",
             coef=False),
        # the operator of the pressure solve on one GPU's share of a convection box
        dict(name="ax_slab32_n7", op="ax", mesh="slab", nx=32, ny=32, nz=16, N=7, dtype="fp64",
             coef=False),
        # the operator as FP32 preconditioners and refinement apply it, at the largest order of
        # the convection runs, on a mesh of odd counts
        dict(name="ax_layers23_n9_fp32", op="ax", mesh="layers", nx=23, ny=25, nz=21, N=9,
             dtype="fp32", coef=False),
        # both gradients of the variable-coefficient operator
        dict(name="ax_backward_cube16_n7", op="ax_backward", mesh="cube", nx=16, ny=16, nz=16,
             N=7, dtype="fp64", coef=True),
        # a right-hand side: mass matrix, direct-stiffness summation, Dirichlet mask
        dict(name="rhs_slab37_n5", op="rhs", mesh="slab", nx=37, ny=29, nz=23, N=5, dtype="fp64",
             coef=False),
        # the convective term of one time step: temperature and velocity, 3/2 rule
        dict(name="advect4_slab32_n7", op="advect", mesh="slab", nx=32, ny=32, nz=16, N=7,
             dtype="fp64", rule="dealias", nf=4, coef=False),
        # the same for one field in FP32 at the lowest order of the convection runs
        dict(name="advect1_cube21_n5_fp32", op="advect", mesh="cube", nx=21, ny=19, nz=23, N=5,
             dtype="fp32", rule="dealias", nf=1, coef=False),
        # a small Poisson solve: a few hundred short iterations
        dict(name="pcg_cube4_n7", op="solve", mesh="cube", nx=4, ny=4, nz=4, N=7, dtype="fp64",
             precond="jacobi", iters=0, coef=False),
        # the headline solve: 100 Jacobi-PCG iterations on the convection box
        dict(name="pcg100_slab32_n7", op="solve", mesh="slab", nx=32, ny=32, nz=16, N=7,
             dtype="fp64", precond="jacobi", iters=100, coef=False),
        # mixed precision with the constant null space: FP64 CG, FP32 Chebyshev preconditioner
        dict(name="cheb_layers12_n9", op="solve", mesh="layers", nx=12, ny=12, nz=12, N=9,
             dtype="fp64", precond="chebyshev", iters=0, coef=False),
        # the pressure solve as a time step runs it: p-multigrid, FP32 cycle
        dict(name="pmg_slab32_n7", op="solve", mesh="slab", nx=32, ny=32, nz=16, N=7,
             dtype="fp64", precond="pmg", iters=0, coef=False),
        # a gradient step through the variable-coefficient Helmholtz solve
        dict(name="grad_cube16_n7", op="grad", mesh="cube", nx=16, ny=16, nz=16, N=7,
             dtype="fp64", precond="jacobi", iters=0, coef=True),
    ]


def _shape(rng, points, N):
    """An element lattice of about `points` local points, sides at least 3."""
    E = max(27.0, points / (N + 1) ** 3)
    fx, fy = math.exp(rng.uniform(-0.35, 0.35)), math.exp(rng.uniform(-0.35, 0.35))
    nx = max(3, round(E ** (1 / 3) * fx))
    ny = max(3, round(E ** (1 / 3) * fy))
    nz = max(3, int(E / (nx * ny)))
    return nx, ny, nz


def draw(rng):
    op = rng.choice(["ax", "ax", "ax_backward", "rhs", "advect", "advect", "solve", "solve",
                     "solve", "grad"])
    c = dict(op=op, mesh=rng.choice(["cube", "slab", "layers"]), dtype="fp64", coef=False)
    lg = rng.uniform
    if op in ("ax", "rhs"):
        c["N"] = rng.randint(3, 10)
        c["dtype"] = rng.choice(["fp64", "fp64", "fp32"])
        c["coef"] = op == "ax" and rng.random() < 0.3
        points = math.exp(lg(math.log(2e4), math.log(8e6)))
    elif op == "ax_backward":
        c["N"] = rng.randint(4, 9)
        c["coef"] = True
        points = math.exp(lg(math.log(2e4), math.log(4e6)))
    elif op == "advect":
        c["N"] = rng.randint(4, 9)
        c["dtype"] = rng.choice(["fp64", "fp32"])
        c["rule"] = rng.choice(["dealias", "dealias", "collocation"])
        c["nf"] = rng.choice([1, 3, 4])
        points = math.exp(lg(math.log(2e4), math.log(5e6)))
    elif op == "solve":
        c["N"] = rng.randint(5, 9)
        c["precond"] = rng.choice(["jacobi", "jacobi", "chebyshev", "pmg", "pmg"])
        c["iters"] = 0
        points = math.exp(lg(math.log(2e4), math.log(2e6)))
        if c["precond"] == "jacobi" and points > 2e5:
            c["iters"] = rng.randint(30, 100)
    else:
        c["N"] = rng.randint(5, 8)
        c["mesh"] = "cube"
        c["precond"] = rng.choice(["jacobi", "pmg"])
        c["iters"] = 0
        c["coef"] = True
        points = math.exp(lg(math.log(2e4), math.log(1e6)))
    c["nx"], c["ny"], c["nz"] = _shape(rng, points, c["N"])
    return c


# ------------------------------------------------------------------ inputs

def _gll(N):
    """GLL nodes, weights and derivative matrix (numpy, 64 bits)."""
    leg = np.polynomial.legendre
    c = np.zeros(N + 1)
    c[N] = 1.0
    x = np.sort(np.real(leg.legroots(leg.legder(c)))) if N > 1 else np.zeros(0)
    d1, d2 = leg.legder(c), leg.legder(c, 2)
    for _ in range(3):  # Newton steps on P_N'
        if N > 1:
            x = x - leg.legval(x, d1) / leg.legval(x, d2)
    x = np.concatenate([[-1.0], 0.5 * (x - x[::-1]), [1.0]])
    w = 2.0 / (N * (N + 1) * leg.legval(x, c) ** 2)
    return x, w, _lagrange(x, x)[1]


def _lagrange(x, y):
    """Values and derivatives at y of the Lagrange polynomials of the nodes x."""
    n, m = len(x), len(y)
    J, D = np.zeros((m, n)), np.zeros((m, n))
    for i in range(n):
        others = [j for j in range(n) if j != i]
        scale = np.prod([x[i] - x[j] for j in others])
        for a in range(m):
            d = [y[a] - x[j] for j in others]
            J[a, i] = np.prod(d) / scale
            D[a, i] = sum(np.prod(d[:s] + d[s + 1:]) for s in range(n - 1)) / scale
    return J, D


def _layers(n, ratio=20.0):
    """n + 1 heights in [0, 1], tanh-clustered to both ends."""
    m = np.arange(n + 1)

    def heights(g):
        return 0.5 * (1.0 + np.tanh(g * (2.0 * m / n - 1.0)) / np.tanh(g))

    lo, hi = 1e-3, 10.0
    for _ in range(100):
        g = 0.5 * (lo + hi)
        d = np.diff(heights(g))
        lo, hi = (g, hi) if d.max() / d.min() < ratio else (lo, g)
    return heights(lo)


def _describe(kind, nx, ny, nz, N):
    """(xyz (E, P, 3) on the GPU, gid (E, P), dirichlet (E, P) or None, n_unique)."""
    f8 = dict(dtype=torch.float64, device=DEV)
    n1, E = N + 1, nx * ny * nz
    lengths = (4.0, 4.0, 1.0) if kind == "slab" else (1.0, 1.0, 1.0)
    xi = _gll(N)[0]
    v = [np.linspace(0.0, L, n + 1) for L, n in zip(lengths, (nx, ny, nz))]
    if kind != "cube":
        v[2] = _layers(nz) if nz > 2 else v[2]
    V = np.stack(np.meshgrid(v[2], v[1], v[0], indexing="ij")[::-1], axis=-1)  # [z][y][x][3]
    if kind == "cube":
        h = np.array([1.0 / nx, 1.0 / ny, 1.0 / nz])
        move = np.random.default_rng(1).uniform(-0.05, 0.05, V.shape) * h
        V[1:-1, 1:-1, 1:-1] += move[1:-1, 1:-1, 1:-1]
    V = torch.tensor(V, **f8)
    l1 = torch.tensor(np.stack([(1.0 - xi) / 2.0, (1.0 + xi) / 2.0]), **f8)
    X = torch.zeros(nz, ny, nx, n1, n1, n1, 3, **f8)
    for a in range(2):
        for b in range(2):
            for c in range(2):
                w = l1[a][:, None, None] * l1[b][None, :, None] * l1[c][None, None, :]
                X += (V[a:a + nz, b:b + ny, c:c + nx][:, :, :, None, None, None, :]
                      * w[..., None])
    if kind != "cube":
        p1, p2 = np.random.default_rng(1).uniform(0.0, 2.0 * np.pi, size=2)
        x, y, z = X[..., 0].clone(), X[..., 1].clone(), X[..., 2]
        sz = torch.sin(math.pi * z)
        dx = 0.15 * lengths[0] / nx * torch.sin(2 * math.pi * y / lengths[1] + p1) * sz
        dy = 0.15 * lengths[1] / ny * torch.sin(2 * math.pi * x / lengths[0] + p2) * sz
        if kind == "layers":
            dx, dy = dx * torch.sin(math.pi * x), dy * torch.sin(math.pi * y)
        X[..., 0], X[..., 1] = x + dx, y + dy
    xyz = X.reshape(E, n1 ** 3, 3)
    side, at = [], []
    for d, n in enumerate((nx, ny, nz)):
        g = torch.arange(n, device=DEV)[:, None] * N + torch.arange(n1, device=DEV)[None, :]
        wrap = kind == "slab" and d < 2
        side.append(n * N + (0 if wrap else 1))
        at.append(g % (n * N) if wrap else g)
    gx = at[0].view(1, 1, nx, 1, 1, n1)
    gy = at[1].view(1, ny, 1, 1, n1, 1)
    gz = at[2].view(nz, 1, 1, n1, 1, 1)
    gid = (gx + side[0] * (gy + side[1] * gz)).reshape(E, n1 ** 3)
    wall = None
    if kind != "layers":
        wall = ((gz == 0) | (gz == nz * N)).expand(nz, ny, nx, n1, n1, n1).clone()
        if kind == "cube":
            wall |= (gx == 0) | (gx == nx * N) | (gy == 0) | (gy == ny * N)
        wall = wall.reshape(E, n1 ** 3)
    return xyz, gid, wall, side[0] * side[1] * side[2]


def _mesh_key(c):
    return c["mesh"], c["nx"], c["ny"], c["nz"], c["N"]


@lru_cache(maxsize=1)
def _mesh(key, extra):
    """The mesh handle that a program sets up once and keeps; `extra` names
    what else it sets up with it (the multigrid levels or an advection rule)."""
    xyz, gid, wall, _ = _describe(*key)
    M = sem.Mesh(xyz.cpu().numpy(), gid.cpu().numpy(),
                 None if wall is None else wall.to(torch.uint8).cpu().numpy(), key[4])
    if extra == "pmg":
        M.setup_pmg()
    elif extra:
        M.setup_advection(extra)
    return M


def _wave(xyz, gen, ell, modes=16):
    """A smooth random field of unit variance at the nodes (E, P)."""
    f8 = dict(dtype=torch.float64, device=DEV)
    kappa = torch.randn(modes, 3, generator=gen, **f8) / (2 * math.pi * ell)
    phi = torch.rand(modes, generator=gen, **f8) * 2 * math.pi
    g = torch.zeros(xyz.shape[:2], **f8)
    for m in range(modes):
        g += torch.cos(2 * math.pi * (xyz * kappa[m]).sum(-1) + phi[m])
    return g * math.sqrt(2.0 / modes)


def _inputs(c, seed, xyz, gid, wall, n_unique):
    """The vectors of a pass, made from the seed alone (a dict of GPU tensors)."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    dt = torch.float64 if c["dtype"] == "fp64" else torch.float32
    f8 = dict(dtype=torch.float64, device=DEV)

    def nodal():
        """One normal number per global node, 0 at walls, at every local point."""
        b = torch.randn(n_unique, generator=gen, **f8)
        if wall is not None:
            b[gid[wall]] = 0.0
        return b[gid]

    v = {}
    if c["coef"]:
        v["k"] = torch.exp(0.5 * _wave(xyz, gen, 0.2)).to(dt)
    if c["op"] == "ax":
        v["u"] = nodal().to(dt)
    elif c["op"] == "ax_backward":
        v["u"] = nodal()
        v["wbar"] = nodal()
    elif c["op"] == "rhs":
        v["f"] = _wave(xyz, gen, 0.25).to(dt)
    elif c["op"] == "advect":
        v["u"] = torch.stack([_wave(xyz, gen, 0.25, 8) for _ in range(3)]).to(dt)
        v["f"] = torch.stack([_wave(xyz, gen, 0.25, 8) for _ in range(c["nf"])]).to(dt)
        if c["nf"] == 1:
            v["f"] = v["f"][0].contiguous()
    else:
        v["b"] = nodal()
        if wall is None:
            v["b"] -= v["b"].mean()
        if c["op"] == "grad":
            v["xbar"] = nodal()
    return v


def _h2(c):
    return 1.0 if c["coef"] else 0.0


def prepare(case, seed):
    extra = ""
    if case.get("precond") == "pmg":
        extra = "pmg"
    elif case["op"] == "advect":
        extra = case["rule"]
    M = _mesh(_mesh_key(case), extra)
    s = _inputs(case, seed, *_describe(*_mesh_key(case)))
    s["mesh"], s["case"] = M, case
    return s


def _solve_opts(c):
    o = dict(precond=c["precond"])
    if c["precond"] == "chebyshev":
        o["precond_prec"] = "fp32"
    return o


def run(state):
    c, M = state["case"], state["mesh"]
    op, k, h2 = c["op"], state.get("k"), _h2(c)
    if op == "ax":
        return sem.ax(M, state["u"], k=k, h2=h2)
    if op == "ax_backward":
        return sem.ax_backward(M, state["u"], state["wbar"], k=k, h2=h2)
    if op == "rhs":
        return sem.mask(M, sem.gs(M, sem.mass(M, state["f"])))
    if op == "advect":
        return sem.advect(M, state["u"], state["f"], rule=c["rule"])
    if op == "solve":
        fixed = c["iters"] > 0
        x, _ = sem.solve(M, state["b"], k=k, h2=h2, rtol=1e-12, fixed_iters=fixed,
                         max_iter=c["iters"] if fixed else 20000, **_solve_opts(c))
        return x
    k = k.detach().requires_grad_()
    b = state["b"].detach().requires_grad_()
    x = sem_solve(M, b, k=k, h2=h2, **_solve_opts(c))
    kbar, bbar = torch.autograd.grad(x, (k, b), state["xbar"])
    return x.detach(), kbar, bbar


# ------------------------------------------------------------------- work

# Nominal iterations of a solve to 1e-12, by preconditioner: what the work of a
# solve is counted with (the count that a mesh takes is its own).
_LEAST = {"jacobi": 200, "chebyshev": 200, "pmg": 10}


def work(case):
    """Bytes that have to cross the memory at least once and flops of the
    contractions.  The geometry counts as what describes it: the coordinates
    of the nodes, or the eight corners where the elements are straight-edged."""
    N = case["N"]
    n1 = N + 1
    E = case["nx"] * case["ny"] * case["nz"]
    nL = E * n1 ** 3
    size = 8 if case["dtype"] == "fp64" else 4
    straight = case["mesh"] == "cube"
    geo = size * (24 * E if straight else 3 * nL)
    vec = size * nL
    apply_flops = nL * (12 * n1 + 18)
    op, coef = case["op"], 1 if case["coef"] else 0
    if op == "ax":
        return {"bytes": geo + (2 + coef) * vec, "flops": apply_flops}
    if op == "ax_backward":
        return {"bytes": geo + 5 * vec, "flops": 2 * apply_flops}
    if op == "rhs":
        return {"bytes": geo + 2 * vec, "flops": 2 * nL}
    if op == "advect":
        q = (3 * n1) // 2 if case["rule"] == "dealias" else n1
        nf = case["nf"]
        up = 2 * (n1 * n1 * n1 * q + n1 * n1 * q * q + n1 * q ** 3)  # one field to the points
        down = up
        return {"bytes": geo + (3 + 2 * nf) * vec,
                "flops": E * (3 * up + nf * (3 * up + down) + q ** 3 * (15 + 5 * nf))}
    iters = case["iters"] or _LEAST[case["precond"]]
    # per iteration: the operator (geometry, direction in, product out) and the
    # vectors x, r, p, read and written, and the diagonal
    n = E * N ** 3
    sweeps = 1 if case["precond"] == "jacobi" else 3 if case["precond"] == "chebyshev" else 12
    one = geo + coef * vec + 2 * 8 * n + 7 * 8 * n
    total = {"bytes": iters * (one + (sweeps - 1) * (geo + 16 * n) / 2),
             "flops": iters * sweeps * apply_flops}
    if op == "grad":
        total = {"bytes": 2 * total["bytes"] + 4 * vec, "flops": 2 * total["flops"]}
    return total


# ------------------------------------------------------------------ exact

def _along(A, u, d):
    """A (m, n) applied along direction d (0 = i, fastest) of u (E, nk, nj, ni)."""
    ax = 3 - d
    t = u.movedim(ax, 3).contiguous()
    return torch.matmul(t, A.t().contiguous()).movedim(3, ax).contiguous()


class _Exact:
    """The discretisation in plain torch, 64 bits."""

    def __init__(self, c):
        self.c, self.N = c, c["N"]
        self.n1 = self.N + 1
        self.xyz, self.gid, self.wall, self.n_unique = _describe(*_mesh_key(c))
        x, w, D = _gll(self.N)
        f8 = dict(dtype=torch.float64, device=DEV)
        self.D = torch.tensor(D, **f8)
        self.Dt = self.D.t().contiguous()
        w = torch.tensor(w, **f8)
        self.w3 = (w[:, None, None] * w[None, :, None] * w[None, None, :])
        self.shape = (self.xyz.shape[0], self.n1, self.n1, self.n1)

    def cube(self, u):
        return u.reshape(self.shape)

    def factors(self, J=None, Dm=None, part=slice(None)):
        """dx_d/dr_a as [a][d] at the nodes, or at points through J (values) and Dm."""
        out = [[None] * 3 for _ in range(3)]
        for d in range(3):
            x = self.xyz[part, :, d].reshape(-1, self.n1, self.n1, self.n1)
            for a in range(3):
                y = x
                for e in range(3):
                    if e == a:
                        y = _along(self.D if Dm is None else Dm, y, e)
                    elif J is not None:
                        y = _along(J, y, e)
                out[a][d] = y
        return out

    @staticmethod
    def adjugate(X):
        """(adj[a][d] = detJ dr_a/dx_d, detJ)."""
        adj = [[None] * 3 for _ in range(3)]
        for a in range(3):
            b, c = (a + 1) % 3, (a + 2) % 3
            for d in range(3):
                e, f = (d + 1) % 3, (d + 2) % 3
                adj[a][d] = X[b][e] * X[c][f] - X[b][f] * X[c][e]
        return adj, X[0][0] * adj[0][0] + X[0][1] * adj[0][1] + X[0][2] * adj[0][2]

    def metric(self):
        adj, det = self.adjugate(self.factors())
        self.B = self.w3 * det
        self.G = {}
        for a in range(3):
            for b in range(a, 3):
                self.G[a, b] = self.G[b, a] = self.w3 / det * sum(
                    adj[a][d] * adj[b][d] for d in range(3))
        return self

    def grad(self, u):
        return [_along(self.D, u, a) for a in range(3)]

    def apply(self, u, k, h2):
        g = self.grad(u)
        w = h2 * self.B * u
        for a in range(3):
            v = sum(self.G[a, b] * g[b] for b in range(3))
            w = w + _along(self.Dt, v if k is None else k * v, a)
        return w

    def kbar(self, u, wb):
        g, q = self.grad(u), self.grad(wb)
        return sum(q[a] * self.G[a, b] * g[b] for a in range(3) for b in range(3))

    def sum_copies(self, v):
        s = torch.zeros(self.n_unique, dtype=torch.float64, device=DEV)
        s.index_add_(0, self.gid.reshape(-1), v.reshape(-1))
        return s

    def diagonal(self, k, h2):
        one = 1.0 if k is None else k
        D2 = (self.D ** 2).t().contiguous()
        d = h2 * self.B
        for a in range(3):
            d = d + _along(D2, one * self.G[a, a], a)
        dd = torch.diagonal(self.D)
        at = [dd.view(1, 1, 1, -1), dd.view(1, 1, -1, 1), dd.view(1, -1, 1, 1)]
        for a in range(3):
            for b in range(a + 1, 3):
                d = d + 2.0 * at[a] * at[b] * one * self.G[a, b]
        return self.sum_copies(d)

    def setup_solve(self, k, h2):
        self.k, self.h2 = k, h2
        self.free = torch.ones(self.n_unique, dtype=torch.float64, device=DEV)
        if self.wall is not None:
            self.free[self.gid[self.wall]] = 0.0
        self.dinv = self.free / self.diagonal(k, h2)
        self.null = self.wall is None and h2 == 0.0

    def solve(self, b, iters, rtol=1e-14, most=20000):
        """CG on the unique nodes: `iters` iterations, or to rtol."""
        if self.null:
            b = b - b.mean()
        x, r = torch.zeros_like(b), b * self.free
        z = self.dinv * r
        p, rho = z.clone(), torch.dot(r, z)
        stop = rtol * float(torch.linalg.norm(r))
        for it in range(iters or most):
            w = self.free * self.sum_copies(self.apply(self.cube(p[self.gid]), self.k, self.h2))
            if self.null:
                w = w - w.mean()
            alpha = rho / torch.dot(p, w)
            x += alpha * p
            r -= alpha * w
            if not iters and it % 10 == 9 and float(torch.linalg.norm(r)) <= stop:
                break
            z = self.dinv * r
            rho, old = torch.dot(r, z), rho
            p = z + rho / old * p
        return x - x.mean() if self.null else x

    def advect(self, u, f, rule):
        if rule == "dealias":
            q = (3 * self.n1) // 2
            y, wq = np.polynomial.legendre.leggauss(q)
            J, Dm = _lagrange(_gll(self.N)[0], y)
            f8 = dict(dtype=torch.float64, device=DEV)
            J, Dm, wq = (torch.tensor(t, **f8) for t in (J, Dm, wq))
            w3 = wq[:, None, None] * wq[None, :, None] * wq[None, None, :]
        else:
            J, Dm, w3 = None, self.D, self.w3

        def to(v):
            for e in range(3):
                v = v if J is None else _along(J, v, e)
            return v

        out = torch.empty_like(f)
        step = 2048
        for e0 in range(0, self.shape[0], step):
            part = slice(e0, e0 + step)
            adj, _ = self.adjugate(self.factors(J, Dm, part))
            uq = [to(u[d, part].reshape(-1, *self.shape[1:])) for d in range(3)]
            V = [w3 * sum(adj[a][d] * uq[d] for d in range(3)) for a in range(3)]
            for m in range(f.shape[0]):
                v = f[m, part].reshape(-1, *self.shape[1:])
                acc = 0.0
                for a in range(3):
                    g = v
                    for e in range(3):
                        g = _along(Dm, g, e) if e == a else g if J is None else _along(J, g, e)
                    acc = acc + V[a] * g
                for e in range(3):
                    acc = acc if J is None else _along(J.t().contiguous(), acc, e)
                out[m, part] = acc.reshape(-1, self.n1 ** 3)
        return out


def exact(case, seed):
    X = _Exact(case)
    v = {n: t.double() for n, t in _inputs(case, seed, X.xyz, X.gid, X.wall, X.n_unique).items()}
    op, h2 = case["op"], _h2(case)
    flat = (X.shape[0], X.n1 ** 3)
    k = X.cube(v["k"]) if case["coef"] else None
    if op == "advect":
        f = v["f"] if v["f"].dim() == 3 else v["f"][None]
        out = X.advect(v["u"], f, case["rule"])
        return out if v["f"].dim() == 3 else out[0]
    X.metric()
    if op == "ax":
        return X.apply(X.cube(v["u"]), k, h2).reshape(flat)
    if op == "ax_backward":
        u, wb = X.cube(v["u"]), X.cube(v["wbar"])
        return X.apply(wb, k, h2).reshape(flat), X.kbar(u, wb).reshape(flat)
    if op == "rhs":
        b = X.sum_copies(X.B * X.cube(v["f"]))[X.gid]
        return b if X.wall is None else b.masked_fill(X.wall, 0.0)
    X.setup_solve(k, h2)
    mult = X.sum_copies(torch.ones(X.shape, dtype=torch.float64, device=DEV))
    x = X.solve(X.sum_copies(v["b"]) / mult, case["iters"])
    if op == "solve":
        return x[X.gid]
    lam = X.solve(X.free * X.sum_copies(v["xbar"]), 0)
    kbar = -X.kbar(X.cube(x[X.gid]), X.cube(lam[X.gid]))
    return x[X.gid], kbar.reshape(flat), (lam / mult)[X.gid]
