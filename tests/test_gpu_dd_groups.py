"""Double-double passes at each workgroup size of dd_lines: one wave, two waves and
four, with a partial last workgroup on the strided axes.  Against the quad oracle,
to the tolerance of the other double-double tests."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from oracle import reference as R

pytestmark = pytest.mark.gpu

TOL_DD = 1e-30


@pytest.mark.parametrize("kind,N", [
    ("coulomb2d", (64, 64)),       # 32 row pairs and 65 lines of 128: one wave each
    ("coulomb2d", (16, 512)),      # 513 lines of 32: one wave (8 lines), partial last group
    ("coulomb3d", (8, 32, 512)),   # 32832 lines of 16 in the fused pass: two waves
    ("coulomb3d", (8, 64, 512)),   # 65664: four waves, 4104 lines of 128 on axis 1: two
    ("coulomb3d", (32, 32, 32)),   # 2112 lines of 64 in the fused pass: one
])
def test_parity_dd_group_sizes(kind, N):
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
