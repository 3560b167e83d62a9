"""Passes B, C and D of small planes in one launch (fsa_plane.hpp): fsa_apply takes
it on 3D grids with N_0 N_1 <= 2048, fsa_apply_events runs the passes apart.  The two
agree bit for bit, at the smallest and the largest planes, with partial teams (axes
of 3 * 2^a, fewer lines than teams) and one more than a whole number of bins; a
choice of another radix family goes back to separate launches; small oracle checks
hold both."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2504_19410_amd import synth
from parity import check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_19410_amd import fsa
    fsa.tune_reset()
    yield fsa
    fsa.tune_reset()


def apart(plan, rho):
    return plan.apply_events(rho, torch.empty_like(rho), [None] * (2 * len(plan.launches())))


def density(L, N, seed):
    rng = synth.SplitMix64(seed)
    gs = synth.draw_gaussians(rng, 3, 3, [-l / 4 for l in L], [l / 4 for l in L],
                              [l / 5 for l in L], [l / 3 for l in L], isotropic=False)
    return synth.eval_gaussians(gs, L, N)


SIZES = [(8, 8, 8), (8, 12, 16), (12, 8, 24), (16, 128, 8), (128, 16, 12), (24, 64, 16),
         (64, 24, 8), (48, 32, 16), (32, 48, 24), (32, 64, 64), (64, 32, 12), (8, 128, 8),
         (96, 16, 8), (16, 96, 8), (128, 8, 16), (32, 32, 32)]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("N", SIZES)
def test_one_launch_equals_separate_launches(F, N, prec):
    L = tuple(0.25 * n for n in N)
    plan = F.Plan("coulomb3d", L, N, prec, eps=0.5).build()
    rho = torch.from_numpy(density(L, N, sum(N))).to(F.DTYPES[prec]).cuda()
    # nothing is read before it is written, in either schedule
    ws = torch.full((plan.workspace_bytes + 256,), 0xff, dtype=torch.uint8, device="cuda")
    phi = plan.apply(rho, workspace=ws)
    ref = apart(plan, rho)
    torch.cuda.synchronize()
    assert torch.equal(phi, ref)
    check(phi.double().cpu().numpy(),
          O.solve("coulomb3d", L, N, rho.double().cpu().numpy(), eps=0.5), prec, f"{N} {prec}")
    inplace = rho.clone()
    plan.apply(inplace, out=inplace, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(inplace, phi)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_other_choices_run_apart(F, prec):
    N, L = (64, 32, 16), (4.0, 2.0, 1.0)
    plan = F.Plan("yukawa3d", L, N, prec, lam=1.0).build()
    rho = torch.from_numpy(density(L, N, 5)).to(F.DTYPES[prec]).cuda()
    base = plan.apply(rho)
    for var in F.tune_variants(prec, "conv", 128):
        F.tune_set(prec, "conv", 128, var, 0)
        a, b = plan.apply(rho), apart(plan, rho)
        torch.cuda.synchronize()
        assert torch.equal(a, b), var
    F.tune_reset()
    F.tune_set_slabs(prec, N, 3)
    c = plan.apply(rho)
    torch.cuda.synchronize()
    F.tune_reset()
    assert torch.equal(c, base)
    plan.autotune(rho, reps=2)
    a, b = plan.apply(rho), apart(plan, rho)
    torch.cuda.synchronize()
    F.tune_reset()
    assert torch.equal(a, b)


def test_dipole_dipole_on_small_planes(F):
    N, L = (32, 24, 48), (4.0, 3.0, 6.0)
    plan = F.Plan("ddi3d", L, N, "f64", n=(0.8, 0.4, -0.4), m=(0.3, 0.9, -0.2)).build()
    rho = torch.from_numpy(density(L, N, 9)).cuda()
    a, b = plan.apply(rho), apart(plan, rho)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and bool(torch.isfinite(a).all())
    assert float(a.abs().max()) > 0.0 and np.isfinite(float(a.sum()))
