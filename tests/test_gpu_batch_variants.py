"""Batches on either side of the bounds of the untuned choices: the real passes, FP64 at
768, change from variant 3 to 0 where the workgroups (4 rows each) no longer have a CU
each; pass B, FP32 at 768, from variant 1 to 3 at 2^15 lines.  A batch chooses by all
its rows together and each problem by its own, and both compute the same bits."""
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


def density(L, N, seed):
    rng = synth.SplitMix64(seed)
    gs = synth.draw_gaussians(rng, len(N), 3, [-l / 4 for l in L], [l / 4 for l in L],
                              [l / 5 for l in L], [l / 3 for l in L], isotropic=False)
    return synth.eval_gaussians(gs, L, N)


def problem(F, kind, N, prec, seed):
    L = tuple(0.25 * n for n in N)
    plan = F.Plan(kind, L, N, prec, eps=0.5).build()
    return plan, torch.from_numpy(density(L, N, seed)).to(F.DTYPES[prec]).cuda()


@pytest.mark.parametrize("rows,alone,batched", [
    ((96, 192), 3, 3),            # 288 rows: variant 3 in both
    ((384, 384, 384), 3, 0),      # 1152 rows together
    ((1536, 48), 0, 0),           # one already beyond the bound, the other not
])
def test_batch_equals_solo_real_passes_768(F, rows, alone, batched):
    assert F.tune_get("f64", "r2c", 768, rows[0])[0] == alone
    assert F.tune_get("f64", "batched_c2r", 768, sum(rows))[0] == batched
    plans, rhos = zip(*[problem(F, "log2d", (n, 768), "f64", 7 + i) for i, n in enumerate(rows)])
    solo = [p.apply(r) for p, r in zip(plans, rhos)]
    outs = F.apply_batched(plans, rhos)
    torch.cuda.synchronize()
    for a, b in zip(solo, outs):
        assert torch.equal(a, b)
    p, r = plans[-1], rhos[-1]
    check(outs[-1].cpu().numpy(), O.solve("log2d", p.L, p.N, r.cpu().numpy(), eps=p.eps), "f64",
          f"batched {p.N}")


@pytest.mark.parametrize("Ns,alone,batched", [
    ([(64, 384, 256), (64, 384, 256)], 1, 3),    # 2 x 16448 lines
    ([(8, 384, 12), (24, 384, 16)], 1, 1),
    ([(128, 384, 256), (12, 384, 8)], 3, 3),     # 32896 lines alone
])
def test_batch_equals_solo_pass_b_768(F, Ns, alone, batched):
    lines = [N[0] * (N[2] + 1) for N in Ns]
    assert F.tune_get("f32", "fwd_t", 768, lines[0])[0] == alone
    assert F.tune_get("f32", "batched_fwd_t", 768, sum(lines))[0] == batched
    plans, rhos = zip(*[problem(F, "coulomb3d", N, "f32", 3 + i) for i, N in enumerate(Ns)])
    solo = [p.apply(r) for p, r in zip(plans, rhos)]
    outs = F.apply_batched(plans, rhos)
    torch.cuda.synchronize()
    for a, b in zip(solo, outs):
        assert torch.equal(a, b)
    p, r = plans[-1], rhos[-1]
    if p.N[0] * p.N[2] <= 4096:
        check(outs[-1].double().cpu().numpy(),
              O.solve("coulomb3d", p.L, p.N, r.double().cpu().numpy(), eps=p.eps), "f32",
              f"batched {p.N}")
