"""The Schwarz local solves at every box size against the oracle's V-cycle.

Orders 2..10 give boxes of 5^3..13^3 points: whole and partial tiles of 16
columns, steps of four and rows of 16 in both precisions, and element counts
that leave the last workgroup partly empty.  Two levels, so the V-cycle is
smoothing on the order under test and the coarsest level's solve.
Tolerances as for the other V-cycles: FP64 1e-12, FP32 2e-4 relative.
"""

import numpy as np
import pytest
import torch

import oracle
from oracle.pmg import PMG
from sem_inputs import box_mesh

pytestmark = pytest.mark.gpu

sem = pytest.importorskip("paper_2501_13240_amd")


@pytest.mark.parametrize("N", range(2, 11))
@pytest.mark.parametrize("shape,dirichlet", [((3, 2, 3), "all"), ((2, 2, 1), "none")])
def test_schwarz_vcycle_every_order(N, shape, dirichlet):
    m = box_mesh(N, shape, (1.0, 1.3, 0.8), dirichlet=dirichlet, jitter=0.05,
                 deform=dict(a=0.1, seed=2, kind="walls"))
    kw = dict(smoother="schwarz", smooth_order=3, coarse_iters=10, orders=(N, 1))
    M = sem.Mesh(m.xyz, m.gid, m.dirichlet, N)
    M.setup_pmg(**kw)
    P0 = oracle.Problem(m.xyz, m.gid, m.dirichlet, N)
    r = np.random.default_rng(N).standard_normal(P0.num.n_free)
    if P0.neumann:
        r -= r.mean()
    rL = torch.tensor(P0.num.to_local(r), dtype=torch.float64, device="cuda")
    out = {p: sem.pmg_apply(M, rL, prec=p).cpu().numpy() for p in ("fp64", "fp32")}
    pmg = PMG(m.xyz, m.gid, m.dirichlet, N, rho=M.pmg_info()[1], **kw)
    ref = P0.num.to_local(pmg.vcycle(r))
    if P0.neumann:
        mean = lambda z: P0.num.from_local_consistent(z).mean()
        ref = ref - mean(ref)
        out = {p: z - mean(z) for p, z in out.items()}
    err = {p: np.linalg.norm(z - ref) / np.linalg.norm(ref) for p, z in out.items()}
    print(f"N={N} {shape} {dirichlet}: fp64 {err['fp64']:.2e} fp32 {err['fp32']:.2e}")
    assert err["fp64"] <= 1e-12
    assert err["fp32"] <= 2e-4
