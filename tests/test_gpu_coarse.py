"""The coarsest multigrid level's resident CG against the oracle's V-cycle.

Sizes at the edges of its workgroups of 256 rows (1, 255, 256, 257 rows, two
workgroups of a singular problem, wrapped columns), a variable coefficient,
and a coarsest level of order 2, which keeps the launch-per-kernel CG.
Tolerances as for the other V-cycles: FP64 differs from the oracle by the
order of the sums only (1e-12 relative after 30 coarse iterations), FP32 2e-4.
"""

import numpy as np
import pytest
import torch

import oracle
from oracle.pmg import PMG
from sem_inputs import box_mesh

pytestmark = pytest.mark.gpu

sem = pytest.importorskip("paper_2501_13240_amd")

CASES = [
    # shape, dirichlet, periodic, orders, rows of the coarsest level
    ((2, 2, 2), "all", (False,) * 3, (2, 1), 1),
    ((4, 6, 18), "all", (False,) * 3, (2, 1), 255),
    ((17, 5, 5), "all", (False,) * 3, (2, 1), 256),
    ((2, 2, 258), "all", (False,) * 3, (2, 1), 257),
    ((7, 7, 6), "none", (False,) * 3, (3, 1), 448),
    ((8, 8, 6), "z", (True, True, False), (2, 1), 320),
    ((4, 4, 3), "z", (True, True, False), (3, 2), 4 * 4 * 4 * 5),
]


@pytest.mark.parametrize("shape,dirichlet,periodic,orders,rows", CASES)
@pytest.mark.parametrize("coef", [False, True])
def test_vcycle_with_resident_coarse_cg(shape, dirichlet, periodic, orders, rows, coef):
    N = orders[0]
    m = box_mesh(N, shape, (1.0, 1.2, 0.9), periodic=periodic, dirichlet=dirichlet, jitter=0.05)
    k = 1.5 + np.sin(3.0 * m.xyz[..., 0]) * np.cos(2.0 * m.xyz[..., 1]) if coef else None
    h2 = 0.5 if coef else 0.0
    M = sem.Mesh(m.xyz, m.gid, m.dirichlet, N)
    M.setup_pmg(orders=orders, smoother="jacobi", smooth_order=3, coarse_iters=30)
    P0 = oracle.Problem(m.xyz, m.gid, m.dirichlet, N, k=k, h2=h2)
    r = np.random.default_rng(rows).standard_normal(P0.num.n_free)
    if P0.neumann:
        r -= r.mean()
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    kd = None if k is None else dev(k)
    out = {p: sem.pmg_apply(M, dev(P0.num.to_local(r)), k=kd, h2=h2, prec=p).cpu().numpy()
           for p in ("fp64", "fp32")}
    pmg = PMG(m.xyz, m.gid, m.dirichlet, N, k=k, h2=h2, rho=M.pmg_info()[1], smoother="jacobi",
              orders=orders, smooth_order=3, coarse_iters=30)
    assert pmg.levels[-1].num.n_free == rows
    ref = P0.num.to_local(pmg.vcycle(r))
    if P0.neumann:
        mean = lambda z: P0.num.from_local_consistent(z).mean()
        ref = ref - mean(ref)
        out = {p: z - mean(z) for p, z in out.items()}
    err = {p: np.linalg.norm(z - ref) / np.linalg.norm(ref) for p, z in out.items()}
    print(f"{shape} {orders} rows {rows} coef {coef}: fp64 {err['fp64']:.2e} fp32 {err['fp32']:.2e}")
    assert err["fp64"] <= 1e-12
    assert err["fp32"] <= 2e-4
