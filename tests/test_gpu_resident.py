"""Jacobi-PCG of a small mesh (one resident kernel) against the oracle's PCG.

Mesh sizes at the edges: one element (no exchange between workgroups), the
largest that stays resident at each order and one element more (launches per
kernel), every order from 5 to 10; Dirichlet, wrapped and singular problems; a
node with more copies than the gather's list holds; more iterations than one
launch runs; the FP32 solves inside a refinement.  Sums differ from the
oracle's in their order only: residual histories over 40 iterations agree to
1e-8 (as for the larger solves), converged solves to a true residual of 1.2e-10
at rtol 1e-10.
"""

import numpy as np
import pytest
import torch

import oracle
from sem_inputs import box_mesh

pytestmark = pytest.mark.gpu

sem = pytest.importorskip("paper_2501_13240_amd")


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def case(N, shape, dirichlet="all", periodic=(False,) * 3, coef=False):
    m = box_mesh(N, shape, (1.0, 1.2, 0.9), periodic=periodic, dirichlet=dirichlet, jitter=0.05)
    k = 1.5 + np.sin(3.0 * m.xyz[..., 0]) * np.cos(2.0 * m.xyz[..., 1]) if coef else None
    return m, m.gid, k, 0.5 if coef else 0.0


def history_and_x(m, gid, k, h2, N, iters=40):
    P = oracle.Problem(m.xyz, gid, m.dirichlet, N, k=k, h2=h2)
    b = np.random.default_rng(N).standard_normal(P.num.n_free)
    if P.neumann:
        b -= b.mean()
    M = sem.Mesh(m.xyz, gid, m.dirichlet, N)
    x, st = sem.solve(M, dev(P.num.to_local(b)), k=None if k is None else dev(k), h2=h2,
                      max_iter=iters, fixed_iters=True, history=True)
    ref = P.solve(b, rtol=1e-30, max_iter=iters, fixed_iters=True)
    np.testing.assert_allclose(st["history"], ref["res_hist"], rtol=1e-8)
    xf = P.num.from_local_consistent(x.cpu().numpy())
    assert np.linalg.norm(xf - ref["x"]) <= 1e-8 * np.linalg.norm(ref["x"])


@pytest.mark.parametrize("N,shape,kw", [
    (5, (8, 6, 4), {}),
    (5, (193, 1, 1), {}),
    (6, (3, 2, 2), dict(dirichlet="none")),
    (7, (2, 2, 2), dict(dirichlet="none", coef=True)),
    (7, (8, 6, 4), dict(dirichlet="z", periodic=(True, True, False))),
    (7, (193, 1, 1), {}),
    (8, (8, 4, 4), dict(coef=True)),
    (9, (4, 4, 4), dict(dirichlet="z", periodic=(True, True, False), coef=True)),
    (10, (4, 4, 4), {}),
    (10, (13, 5, 1), dict(dirichlet="none")),
])
def test_fixed_iterations_match_oracle(N, shape, kw):
    history_and_x(*case(N, shape, **kw), N)


def test_node_with_many_copies():
    """All corners of 20 separate elements are one unknown: 160 copies on
    each of an element's eight corners, of which the list holds some."""
    m, _, k, h2 = case(5, (20, 1, 1), coef=True)
    gid = np.arange(m.E * m.P, dtype=m.gid.dtype).reshape(m.E, m.P)
    c = [i + 6 * j + 36 * l for i in (0, 5) for j in (0, 5) for l in (0, 5)]
    gid[:, c] = gid[0, 0]
    m.dirichlet[...] = 0
    history_and_x(m, gid, k, h2, 5)


@pytest.mark.parametrize("kw", [dict(), dict(mode="mixed_ir")])
def test_one_element(kw):
    """64 unknowns: 40 iterations reach 1e-17 of the start, where the residuals
    of two orders of summation no longer agree; so the converged solve."""
    m, gid, _, _ = case(5, (1, 1, 1))
    P = oracle.Problem(m.xyz, gid, m.dirichlet, 5)
    b = np.random.default_rng(5).standard_normal(P.num.n_free)
    M = sem.Mesh(m.xyz, gid, m.dirichlet, 5)
    x, st = sem.solve(M, dev(P.num.to_local(b)), rtol=1e-10, **kw)
    xf = P.num.from_local_consistent(x.cpu().numpy())
    assert np.linalg.norm(b - P.apply(xf)) <= 1.2e-10 * np.linalg.norm(b)


@pytest.mark.parametrize("kw", [dict(), dict(mode="mixed_ir")])
def test_more_iterations_than_a_launch(kw):
    N = 7
    m, gid, _, _ = case(N, (4, 4, 3), dirichlet="z")
    k = 10.0 ** (4.0 * np.random.default_rng(1).random((m.E, m.P)))
    P = oracle.Problem(m.xyz, gid, m.dirichlet, N, k=k)
    b = np.random.default_rng(0).standard_normal(P.num.n_free)
    M = sem.Mesh(m.xyz, gid, m.dirichlet, N)
    x, st = sem.solve(M, dev(P.num.to_local(b)), k=dev(k), rtol=1e-10, max_iter=20000, **kw)
    print(kw, st["iters"], st["outer_iters"])
    assert st["converged"] == 1 and st["iters"] > 512
    xf = P.num.from_local_consistent(x.cpu().numpy())
    assert np.linalg.norm(b - P.apply(xf)) <= 1.2e-10 * np.linalg.norm(b)
