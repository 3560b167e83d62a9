"""Double-double passes where the lines of a launch do not fill its workgroups:
fewer lines than one workgroup takes (1024 / P), a partial last workgroup on the
strided axes (N_last + 1 lines), and the shortest and longest rows in pairs.
Against the quad oracle, to the tolerance of the other double-double tests."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from oracle import reference as R

pytestmark = pytest.mark.gpu

TOL_DD = 1e-30


@pytest.mark.parametrize("kind,N", [
    ("coulomb3d", (8, 8, 8)),      # 32 row pairs of 64 per workgroup
    ("coulomb3d", (8, 64, 8)),     # 9 bins per plane on axis 1
    ("coulomb2d", (8, 8)),         # one workgroup per pass, mostly empty
    ("coulomb2d", (8, 1024)),      # rows of 2048, one pair per workgroup
    ("coulomb2d", (256, 8)),       # 9 lines of 512, two per workgroup
])
def test_parity_dd_partial_workgroups(kind, N):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_19410_amd import fsa as F
    rng = np.random.default_rng(sum(N))
    rho = np.empty(N + (2,))
    rho[..., 0] = rng.standard_normal(N)
    rho[..., 1] = rho[..., 0] * 2.0 ** -53 * rng.uniform(-1, 1, N)
    L = tuple(0.25 * n for n in N)
    plan = F.Plan(kind, L, N, "dd").build()
    ws = torch.full((plan.workspace_bytes + 256,), 0xff, dtype=torch.uint8, device="cuda")
    phi = plan.apply(torch.from_numpy(rho).cuda(), workspace=ws)   # every entry read is written
    torch.cuda.synchronize()
    ref = O.solve_quad(kind, L, N, rho, plan.eps)
    assert R.dd_rel_l2_err(phi.cpu().numpy(), ref) <= TOL_DD
