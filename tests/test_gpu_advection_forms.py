"""The convective term on straight-edged meshes, whose factors are formed from
the elements' corners (over-integrated from N = 3 on, collocation always),
against the oracle's; one node moved by 1e-9 of its element takes the stored
factors.  Sheared, jittered elements; one field and three.  Tolerances as for the stored factors: FP64
1e-12, FP32 2e-5 of the largest value.
"""

import numpy as np
import pytest
import torch

from oracle.advection import convect
from sem_inputs import box_mesh, random_fourier_field, velocity_field

pytestmark = pytest.mark.gpu

sem = pytest.importorskip("paper_2501_13240_amd")


def dev(a, dtype=torch.float64):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


@pytest.mark.parametrize("curved", [False, True])
@pytest.mark.parametrize("dealias", [True, False])
@pytest.mark.parametrize("N", range(2, 11))
def test_forms_match_oracle(N, dealias, curved):
    m = box_mesh(N, (3, 2, 2), (1.0, 1.3, 0.7), dirichlet="all", jitter=0.2)
    m.xyz[..., 0] += 0.3 * m.xyz[..., 1]
    m.xyz[..., 2] += 0.2 * m.xyz[..., 0]
    if curved:
        m.xyz[0, 1 + (N + 1) + (N + 1) ** 2, 0] += 1e-9  # an element-interior node
    rule = "dealias" if dealias else "collocation"
    u = velocity_field(m.xyz, seed=11)
    f = np.stack([random_fourier_field(m.xyz, seed=s) for s in (7, 8, 9)])
    M = sem.Mesh(m.xyz, m.gid, m.dirichlet, N)
    ref = np.stack([convect(np.moveaxis(u, 0, 2), g, m.xyz, N, dealias=dealias) for g in f])
    for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 2e-5)):
        out = sem.advect(M, dev(u, dtype), dev(f, dtype), rule=rule).double().cpu().numpy()
        one = sem.advect(M, dev(u, dtype), dev(f[1], dtype), rule=rule).double().cpu().numpy()
        err = np.abs(out - ref).max() / np.abs(ref).max()
        print(f"N {N} {rule} curved {curved} {dtype}: {err:.2e}")
        assert err <= tol
        assert np.array_equal(one, out[1])
