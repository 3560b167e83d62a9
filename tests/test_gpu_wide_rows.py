"""Pass B, FP32 at length 768: variant 3 (whole-line tiles of 16) computes bitwise what
variant 1 computes, where its last tile is partial (N_0 = 8, 12, 24) and where it is
whole, and an oracle check holds both; untuned launches choose between the two by
their lines alone.  The same for the real passes, FP64 at 768: variant 3 (twiddles
ahead of the exchanges) against variant 0, where the last tile is partial (its tiles
take 4 rows; 3D planes of 8 and 12) and where workgroups take several."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2504_19410_amd import synth
from parity import check


def density(L, N, seed):
    rng = synth.SplitMix64(seed)
    gs = synth.draw_gaussians(rng, 3, 3, [-l / 4 for l in L], [l / 4 for l in L],
                              [l / 5 for l in L], [l / 3 for l in L], isotropic=False)
    return synth.eval_gaussians(gs, L, N)


def test_untuned_choice():
    from paper_2504_19410_amd import fsa
    fsa.tune_reset()
    assert 3 in fsa.tune_variants("f32", "fwd_t", 768)
    assert 3 not in fsa.tune_variants("f64", "fwd_t", 768)
    for n in (64, 256, 384, 512, 1024, 1536):
        assert 3 not in fsa.tune_variants("f32", "fwd_t", n), n
    assert fsa.tune_get("f32", "fwd_t", 768, (1 << 15) - 1)[0] == 1
    assert fsa.tune_get("f32", "fwd_t", 768, 1 << 15)[0] == 3


@pytest.mark.gpu
@pytest.mark.parametrize("N", [(8, 384, 8), (24, 384, 16), (12, 384, 12), (64, 384, 24)])
def test_variants_agree(N):
    from paper_2504_19410_amd import fsa
    L = tuple(0.25 * n for n in N)
    plan = fsa.Plan("coulomb3d", L, N, "f32", eps=0.5).build()
    rho = torch.from_numpy(density(L, N, sum(N))).float().cuda()
    lines = plan.pass_lines()[[p[0] for p in plan.passes()].index("fwd_t")]
    phi = []
    try:
        for var in (1, 3):
            fsa.tune_set("f32", "fwd_t", 768, var, 0, lines)
            phi.append(plan.apply(rho).clone())
        torch.cuda.synchronize()
    finally:
        fsa.tune_reset()
    assert torch.equal(phi[0], phi[1])
    ref = O.solve("coulomb3d", L, N, rho.double().cpu().numpy(), eps=plan.eps)
    check(phi[1].double().cpu().numpy(), ref, "f32", f"wide rows {N}")


def test_untuned_choice_real_passes():
    from paper_2504_19410_amd import fsa
    fsa.tune_reset()
    for p in ("r2c", "c2r"):
        assert 3 in fsa.tune_variants("f64", p, 768)
        assert 3 not in fsa.tune_variants("f32", p, 768)
        assert 3 not in fsa.tune_variants("f64", p, 1536)
        assert fsa.tune_get("f64", p, 768, 1024)[0] == 3
        assert fsa.tune_get("f64", p, 768, 1025)[0] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("N", [(8, 12, 768), (12, 8, 768), (64, 48, 768)])
def test_real_variants_agree(N):
    from paper_2504_19410_amd import fsa
    L = tuple(0.25 * n for n in N)
    plan = fsa.Plan("coulomb3d", L, N, "f64", eps=0.5).build()
    rho = torch.from_numpy(density(L, N, sum(N))).double().cuda()
    phi = []
    try:
        for var in (0, 3):
            for p in ("r2c", "c2r"):
                fsa.tune_set("f64", p, 768, var, 0, N[0] * N[1])
            phi.append(plan.apply(rho).clone())
        torch.cuda.synchronize()
    finally:
        fsa.tune_reset()
    assert torch.equal(phi[0], phi[1])
    if N[0] * N[1] <= 96:
        ref = O.solve("coulomb3d", L, N, rho.cpu().numpy(), eps=plan.eps)
        check(phi[1].cpu().numpy(), ref, "f64", f"early twiddles {N}")
