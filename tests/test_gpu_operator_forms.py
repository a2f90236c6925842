"""Every form of the matrix-core operator (N >= 5) against the oracle.

Straight-edged meshes form their factors from the elements' corners, curved
ones read stored factors; one node moved by 1e-9 of its element turns the
first kind into the second.  Each is applied alone, with k and h2, backward
(both gradients in one pass), and inside the solves (with the single-copy
nodes split off: Dirichlet and singular, plain and nontemporal shared-copy
stores, FP64 and FP32).
Tolerances: FP64 operator and gradients 1e-12, FP32 2e-6 of the operator's
majorant-free norm (24-bit sums of 3 (N+1) products), solves: true residual by
the oracle's operator 1.2e-10 at rtol 1e-10.
"""

import numpy as np
import pytest
import torch

import oracle
from oracle.operator import local_apply
from sem_inputs import box_mesh

pytestmark = pytest.mark.gpu

sem = pytest.importorskip("paper_2501_13240_amd")


def rel(a, b):
    return np.linalg.norm(np.asarray(a, dtype=np.float64) - b) / np.linalg.norm(b)


def dev(a, dtype=torch.float64):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def mesh(N, curved, dirichlet="all", shape=(3, 2, 2)):
    m = box_mesh(N, shape, (1.0, 1.3, 0.7), dirichlet=dirichlet, jitter=0.2)
    # shear: straight edges, no right angles (a linear map keeps the trilinear form)
    m.xyz[..., 0] += 0.3 * m.xyz[..., 1]
    m.xyz[..., 2] += 0.2 * m.xyz[..., 0]
    if curved:
        P1 = N + 1  # an element-interior node
        m.xyz[0, 1 + P1 + P1 * P1, 0] += 1e-9
    return m


@pytest.mark.parametrize("N", range(5, 11))
@pytest.mark.parametrize("curved", [False, True])
def test_applies_and_gradients(N, curved):
    m = mesh(N, curved)
    M = sem.Mesh(m.xyz, m.gid, m.dirichlet, N)
    rng = np.random.default_rng(N)
    u, wb = rng.standard_normal((2, m.E, m.P))
    k = 1.0 + rng.random((m.E, m.P))
    P = oracle.Problem(m.xyz, m.gid, m.dirichlet, N)
    for kk, h2 in ((None, 0.0), (k, 0.7)):
        ref = local_apply(u, P.G, P.B, N, k=kk, h2=h2)
        kd = None if kk is None else dev(kk)
        k32 = None if kk is None else dev(kk, torch.float32)
        assert rel(sem.ax(M, dev(u), k=kd, h2=h2).cpu().numpy(), ref) <= 1e-12
        assert rel(sem.ax(M, dev(u, torch.float32), k=k32, h2=h2).cpu().numpy(), ref) <= 2e-6
        ub, kb = sem.ax_backward(M, dev(u), dev(wb), k=kd, h2=h2)
        assert rel(ub.cpu().numpy(), local_apply(wb, P.G, P.B, N, k=kk, h2=h2)) <= 1e-12
        assert rel(kb.cpu().numpy(), oracle.kgrad_contraction(u, wb, P.G, N)) <= 1e-12
        # one gradient alone takes the separate kernels
        ub1, none = sem.ax_backward(M, dev(u), dev(wb), k=kd, h2=h2, need_kbar=False)
        assert none is None and rel(ub1.cpu().numpy(), ub.cpu().numpy()) <= 1e-13


@pytest.mark.parametrize("N", range(5, 11))
@pytest.mark.parametrize("curved", [False, True])
@pytest.mark.parametrize("dirichlet", ["all", "none"])
def test_solves(N, curved, dirichlet, store_form):
    m = mesh(N, curved, dirichlet)
    M = sem.Mesh(m.xyz, m.gid, m.dirichlet, N)
    P = oracle.Problem(m.xyz, m.gid, m.dirichlet, N)
    b = np.random.default_rng(N).standard_normal(P.num.n_free)
    if P.neumann:
        b -= b.mean()
    bL = dev(P.num.to_local(b))
    for kw in (dict(), dict(precond="chebyshev", precond_prec="fp64"),
               dict(precond="chebyshev", precond_prec="fp32"), dict(mode="mixed_ir")):
        x, st = sem.solve(M, bL, rtol=1e-10, **kw)
        r = P.project(b) - P.apply(P.num.from_local_consistent(x.cpu().numpy()))
        res = np.linalg.norm(r) / np.linalg.norm(b)
        print(f"N={N} curved={curved} {dirichlet} {kw}: {st['iters']} it, residual {res:.2e}")
        assert st["converged"] == 1 and res <= 1.2e-10
