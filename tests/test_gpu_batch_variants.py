"""Batches on either side of the bounds of the untuned choices: the real passes, FP64 at
768, change from variant 3 to 0 where the workgroups (4 rows each) no longer have a CU
each; pass B, FP32 at 768, from family 0 to 1 at 2^8 lines and within it to variant 3
at 2^15.  A batch chooses by all
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
    ([(8, 384, 12), (12, 384, 8)], 0, 0),        # 104 and 108 lines: the other family
    ([(24, 384, 16), (8, 384, 12)], 1, 1),       # 408 and 104: a launch for each family
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


@pytest.mark.parametrize("prec,Ns,key,families", [
    ("f32", [(64, 512, 16), (256, 512, 64)], ("fwd_t", 1024), (0, 1)),   # 2^14 lines
    ("f64", [(8, 384, 8), (32, 384, 16)], ("inv_t", 768), (0, 1)),       # 2^8
    ("f32", [(8, 384, 8), (16, 384, 24)], ("inv_t", 768), (0, 1)),
    ("f32", [(48, 1024, 64), (96, 1024, 64)], ("inv_t", 2048), (0, 1)),  # 2^12
])
def test_batch_of_both_families(F, prec, Ns, key, families):
    """Problems whose untuned family differs run in launches of their own."""
    plans, rhos = zip(*[problem(F, "coulomb3d", N, prec, 5 + i) for i, N in enumerate(Ns)])
    for N, f in zip(Ns, families):
        assert F.tune_get(prec, *key, N[0] * (N[2] + 1))[0] == f
    solo = [p.apply(r) for p, r in zip(plans, rhos)]
    outs = [torch.empty_like(r) for r in rhos]
    ws = torch.empty(F.batch_workspace_bytes(plans) + 256, dtype=torch.uint8, device="cuda")
    for _ in range(2):                              # captured, then replayed
        F.apply_batched(plans, rhos, outs, ws)
        torch.cuda.synchronize()
        for a, b in zip(solo, outs):
            assert torch.equal(a, b)


@pytest.mark.parametrize("prec,N", [("f32", (128, 512, 128)), ("f64", (128, 512, 128)),
                                    ("f32", (32, 384, 48))])
def test_slabs_keep_the_family(F, prec, N):
    """Slabs whose lines fall below a bound that the whole launch is above."""
    plan, rho = problem(F, "coulomb3d", N, prec, 11)
    try:
        whole = plan.apply(rho).clone()
        for slabs in (2, 5):
            F.tune_set_slabs(prec, N, slabs)
            part = plan.apply(rho)
            torch.cuda.synchronize()
            assert torch.equal(part, whole), slabs
    finally:
        F.tune_reset()
