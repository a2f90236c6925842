"""Every pair of levels of the default hierarchies, whose transfers take a
node's first copy only, and the smoother's fused sums at one, two and three
steps, in a V-cycle against the oracle's (which averages the copies).  Pairs of
sizes outside the hierarchies, and a mesh that identifies nodes whose
interpolated values differ, keep the averaging transfers.  Tolerances as for
the other V-cycles: FP64 1e-12 relative, FP32 2e-4.
"""

import numpy as np
import pytest
import torch

import oracle
from oracle.pmg import PMG, level_orders
from sem_inputs import box_mesh

pytestmark = pytest.mark.gpu

sem = pytest.importorskip("paper_2501_13240_amd")


def check(m, gid, N, orders, **cycle):
    M = sem.Mesh(m.xyz, gid, m.dirichlet, N)
    M.setup_pmg(orders=orders, **cycle)
    P0 = oracle.Problem(m.xyz, gid, m.dirichlet, N)
    r = np.random.default_rng(N).standard_normal(P0.num.n_free)
    rL = torch.tensor(P0.num.to_local(r), dtype=torch.float64, device="cuda")
    z = {p: sem.pmg_apply(M, rL, prec=p).cpu().numpy() for p in ("fp64", "fp32")}
    ref = P0.num.to_local(PMG(m.xyz, gid, m.dirichlet, N, rho=M.pmg_info()[1], orders=orders,
                              **cycle).vcycle(r))
    err = {p: np.linalg.norm(a - ref) / np.linalg.norm(ref) for p, a in z.items()}
    print(f"N {N} {orders} {cycle}: {err['fp64']:.2e} {err['fp32']:.2e}")
    assert err["fp64"] <= 1e-12 and err["fp32"] <= 2e-4


@pytest.mark.parametrize("smoother,order", [("schwarz", 1), ("schwarz", 2), ("schwarz", 3),
                                            ("jacobi", 3)])
@pytest.mark.parametrize("N", range(2, 11))
def test_default_hierarchies(N, smoother, order):
    m = box_mesh(N, (3, 2, 2), (1.0, 1.2, 0.9), dirichlet="z", jitter=0.05)
    check(m, m.gid, N, tuple(level_orders(N)), smoother=smoother, smooth_order=order,
          coarse_iters=10)


@pytest.mark.parametrize("orders", [(7, 5, 1), (6, 5, 4, 1)])
def test_other_pairs(orders):
    m = box_mesh(orders[0], (3, 2, 2), (1.0, 1.2, 0.9), dirichlet="z", jitter=0.05)
    check(m, m.gid, orders[0], orders, smoother="jacobi", smooth_order=3, coarse_iters=10)


def test_copies_that_interpolate_differently():
    N = 5
    m = box_mesh(N, (3, 2, 2), (1.0, 1.2, 0.9), dirichlet="z", jitter=0.05)
    gid = m.gid.copy()
    q = (2 * (N + 1) + 2) * (N + 1) + 2  # an interior node of two elements as one unknown
    gid[5, q] = gid[0, q]
    check(m, gid, N, (5, 2, 1), smoother="jacobi", smooth_order=3, coarse_iters=10)
