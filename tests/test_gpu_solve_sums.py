"""The Jacobi-PCG's reductions of the operator's sums: by every block of the
residual update up to 4096 sums (two an element with the null-space projection),
by a launch of their own above.  Meshes on either side of the line, at orders
with one, two, four and eight wavefronts per element; residual histories of 25
fixed iterations agree with the oracle's to 1e-8 (only the order of the sums
differs), and a solve that stops on the tolerance leaves its last iterate as
the fixed-length solve of as many iterations does.
"""

import numpy as np
import pytest
import torch

import oracle
from sem_inputs import box_mesh

pytestmark = pytest.mark.gpu

sem = pytest.importorskip("paper_2501_13240_amd")


@pytest.mark.parametrize("N,shape,dirichlet", [
    (5, (16, 16, 8), "none"),  # 2048 elements, 4096 sums
    (5, (241, 17, 1), "all"),  # 4097
    (6, (16, 16, 1), "all"),
    (7, (193, 1, 1), "none"),
    (10, (5, 5, 3), "all"),
])
def test_both_sides_match_oracle(N, shape, dirichlet):
    m = box_mesh(N, shape, (1.0, 1.2, 0.9), dirichlet=dirichlet, jitter=0.05)
    P = oracle.Problem(m.xyz, m.gid, m.dirichlet, N)
    b = np.random.default_rng(N).standard_normal(P.num.n_free)
    if P.neumann:
        b -= b.mean()
    M = sem.Mesh(m.xyz, m.gid, m.dirichlet, N)
    bL = torch.tensor(P.num.to_local(b), dtype=torch.float64, device="cuda")
    x, st = sem.solve(M, bL, max_iter=25, fixed_iters=True, history=True)
    ref = P.solve(b, rtol=1e-30, max_iter=25, fixed_iters=True)
    np.testing.assert_allclose(st["history"], ref["res_hist"], rtol=1e-8)
    tol = st["history"][20] / st["history"][0] * (1 + 1e-9)
    x1, st1 = sem.solve(M, bL, rtol=tol)
    x2, st2 = sem.solve(M, bL, max_iter=st1["iters"], fixed_iters=True)
    assert st1["converged"] == 1 and st1["iters"] <= 20 and torch.equal(x1, x2)
