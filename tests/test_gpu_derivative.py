"""The strided launches of the source derivative (fsa_spectral.hip) where their split
can go wrong: sets that are not a multiple of 8, half-spectrum rows that end inside a
group (every length leaves N/2 + 1 bins), the smallest and longest lines (one stage;
groups narrower than 128 bytes), lengths of 3 * 2^a.  Whole evaluations against the
oracle at the parity tests' tolerances, 1e-12 in FP64 and 5e-6 in FP32."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2504_19410_amd import synth
from parity import check

pytestmark = pytest.mark.gpu

DIP_N = (0.82778, 0.41505, -0.37751)
DIP_M = (0.3118, 0.9378, -0.15214)


@pytest.fixture(scope="module")
def F():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_19410_amd import fsa
    return fsa


def density(L, N, seed):
    rng = synth.SplitMix64(seed)
    d = len(N)
    gs = synth.draw_gaussians(rng, d, 3, [-l / 4 for l in L], [l / 4 for l in L],
                              [l / 5 for l in L], [l / 3 for l in L], isotropic=False)
    return synth.eval_gaussians(gs, L, N)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("N", [(8, 8, 8), (12, 24, 16), (24, 12, 8), (8, 96, 12), (384, 8, 8),
                               (8, 768, 8), (1024, 12, 8), (8, 2048, 8), (2048, 8, 8)])
def test_ddi3d(F, N, prec):
    L = tuple(0.25 * n for n in N)
    plan = F.Plan("ddi3d", L, N, prec, eps=0.5, n=DIP_N, m=DIP_M).build()
    rho = torch.from_numpy(density(L, N, sum(N))).to(F.DTYPES[prec]).cuda()
    phi = plan.apply(rho)
    torch.cuda.synchronize()
    ref = O.solve_ddi(L, N, rho.double().cpu().numpy(), plan.eps, DIP_N, DIP_M)
    check(phi.double().cpu().numpy(), ref, prec, f"ddi {N} {prec}")


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("N", [(8, 8), (96, 12), (2048, 8)])
def test_quasi2d(F, N, prec):
    L, n = tuple(0.25 * m for m in N), (0.3, 0.5, np.sqrt(0.66))
    plan = F.Plan("quasi2d_ddi", L, N, prec, eps=0.3, n=n, eta=0.3).build()
    rho = torch.from_numpy(density(L, N, sum(N))).to(F.DTYPES[prec]).cuda()
    phi = plan.apply(rho)
    torch.cuda.synchronize()
    ref = O.solve_q2d(L, N, rho.double().cpu().numpy(), plan.eps, 0.3, n)
    check(phi.double().cpu().numpy(), ref, prec, f"quasi2d {N} {prec}")
