"""Which schedule a small 3D grid takes: the kernels one fsa_apply enqueues, counted in
a captured graph (3 with passes B, C and D in one launch, 5 apart)."""
import ctypes
import os

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_19410_amd import fsa
    fsa.tune_reset()
    yield fsa
    fsa.tune_reset()


def kernels(plan, rho):
    hip = ctypes.CDLL("libamdhip64.so")
    out, ws, s = torch.empty_like(rho), plan.workspace(), torch.cuda.Stream()
    torch.cuda.synchronize()
    st, graph, n = ctypes.c_void_p(s.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t()
    assert hip.hipStreamBeginCapture(st, 1) == 0
    plan.apply(rho, out, workspace=ws, stream=s)
    assert hip.hipStreamEndCapture(st, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return n.value


def make(F, N, prec):
    plan = F.Plan("coulomb3d", tuple(0.25 * n for n in N), N, prec, eps=0.5).build()
    return plan, torch.zeros(N, dtype=F.DTYPES[prec], device="cuda")


@pytest.mark.parametrize("N,prec,want", [
    ((8, 8, 8), "f32", 3), ((32, 32, 32), "f64", 3), ((64, 32, 16), "f64", 3),
    ((16, 128, 8), "f64", 3), ((32, 64, 512), "f32", 3), ((32, 64, 512), "f64", 3),
    # few FP64 planes with a long chain per thread
    ((12, 96, 8), "f64", 5), ((12, 128, 64), "f64", 5), ((96, 16, 48), "f64", 5),
    ((12, 96, 64), "f64", 5), ((24, 64, 48), "f64", 3), ((12, 96, 96), "f64", 3), ((96, 16, 96), "f64", 3),
    ((12, 96, 8), "f32", 3), ((96, 8, 8), "f64", 3),
    # past the plane's size, and an axis longer than 128
    ((48, 48, 8), "f32", 5), ((8, 192, 8), "f32", 5),
])
def test_untuned_schedule(F, N, prec, want):
    plan, rho = make(F, N, prec)
    assert kernels(plan, rho) == want


def arch():
    return torch.cuda.get_device_properties(0).gcnArchName


@pytest.mark.parametrize("N,prec", [((32, 32, 32), "f64"), ((32, 64, 16), "f32")])
def test_a_tuned_decision_is_kept(F, N, prec, tmp_path):
    """A table that says apart runs the passes apart, one that says one launch in one,
    whatever the untuned choice is; the results are the same bits."""
    plan, _ = make(F, N, prec)
    rho = torch.randn(N, dtype=F.DTYPES[prec], device="cuda")
    out = []
    try:
        for one, want in ((0, 5), (1, 3)):
            path = tmp_path / "t.json"
            path.write_text('{"format": "fsa-tune-1", "arch": "%s", "entries": [], "schedules": '
                            '[{"precision": "%s", "grid": [%d, %d, %d], "slabs": 1, '
                            '"one_launch": %d, "us": 1.0}]}' % (arch(), prec, *N, one))
            F.tune_load(str(path))
            assert kernels(plan, rho) == want
            out.append(plan.apply(rho).clone())
        torch.cuda.synchronize()
        assert torch.equal(*out)
    finally:
        F.tune_reset()


@pytest.mark.parametrize("N,prec,want", [((12, 128, 8), "f64", 5), ((16, 16, 16), "f64", 3)])
def test_autotune_keeps_the_faster_schedule(F, N, prec, want):
    """At 12 x 128 x 8 apart is 20% faster, at 16^3 one launch is 25% faster."""
    plan, rho = make(F, N, prec)
    try:
        plan.autotune(torch.randn_like(rho), reps=9)
        assert kernels(plan, rho) == want
    finally:
        F.tune_reset()


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_one_launch_beside_other_choices(F, prec, tmp_path):
    """A grid tuned to one launch keeps it where the entries of its passes, faster
    apart, are of another radix family: fsa_apply, the passes apart and a batch (alone
    or with a problem that follows those entries) give the same bits."""
    N, M = (64, 32, 16), (64, 64, 16)
    plan, _ = make(F, N, prec)
    other, _ = make(F, M, prec)
    rho = torch.randn(N, dtype=F.DTYPES[prec], device="cuda")
    rho2 = torch.randn(M, dtype=F.DTYPES[prec], device="cuda")
    base = plan.apply(rho).clone()
    rows = ", ".join('{"precision": "%s", "pass": "%s", "length": 128, "class": %d, "variant": '
                     '1, "occupancy": 0, "us": 5.0}' % (prec, p, c)
                     for p in ("conv", "fwd_t", "inv_t") for c in range(8, 14))
    path = tmp_path / "t.json"
    path.write_text('{"format": "fsa-tune-1", "arch": "%s", "entries": [%s], "schedules": '
                    '[{"precision": "%s", "grid": [%d, %d, %d], "slabs": 1, "one_launch": 1, '
                    '"us": 1.0}]}' % (arch(), rows, prec, *N))
    try:
        F.tune_load(str(path))
        assert kernels(plan, rho) == 3 and kernels(other, rho2) == 5
        one = plan.apply(rho).clone()
        two = other.apply(rho2).clone()
        apart = plan.apply_events(rho, torch.empty_like(rho), [None] * (2 * len(plan.launches())))
        (alone,) = F.apply_batched([plan], [rho])
        both = F.apply_batched([plan, other], [rho, rho2])
        torch.cuda.synchronize()
        for x in (one, apart, alone, both[0]):
            assert torch.equal(x, base)
        assert torch.equal(both[1], two)
        # set by hand, the other family is what runs
        F.tune_set(prec, "conv", 128, 1, 0, 2 * N[1] * (N[2] + 1))
        assert kernels(plan, rho) == 5
    finally:
        F.tune_reset()


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_autotune_leaves_the_passes_their_fastest(F, prec, tmp_path):
    """The entries of B, C and D name what was fastest for each pass, also where the
    grid was tuned to one launch, and the tuned batch equals the tuned solo run."""
    import json
    N = (32, 32, 64)
    plan, _ = make(F, N, prec)
    rho = torch.randn(N, dtype=F.DTYPES[prec], device="cuda")
    try:
        plan.autotune(rho, reps=5)
        path = tmp_path / "t.json"
        F.tune_save(str(path))
        doc = json.loads(path.read_text())
        assert [r.get("one_launch") for r in doc["schedules"]] == [1]
        assert {e["pass"] for e in doc["entries"]} == {"r2c", "fwd_t", "conv", "inv_t", "c2r"}
        a = plan.apply(rho).clone()
        (b,) = F.apply_batched([plan], [rho])
        torch.cuda.synchronize()
        assert torch.equal(a, b)
    finally:
        F.tune_reset()


SHIPPED = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                       "paper_2504_19410_amd", "tune", "gfx950.json")


@pytest.mark.parametrize("N,prec", [((64, 32, 256), "f64"), ((64, 16, 32), "f64"),
                                    ((128, 16, 16), "f32"), ((16, 128, 64), "f32")])
def test_entries_of_other_grids_do_not_decide(F, N, prec):
    """The shipped table names the other radix family for passes of larger grids, whose
    size class is the nearest one: such grids run in one launch all the same, with the
    bits that the passes give apart."""
    plan, rho = make(F, N, prec)
    rho.normal_()
    try:
        F.tune_load(SHIPPED)
        assert kernels(plan, rho) == 3
        a = plan.apply(rho).clone()
        b = plan.apply_events(rho, torch.empty_like(rho), [None] * (2 * len(plan.launches())))
        torch.cuda.synchronize()
        assert torch.equal(a, b)
    finally:
        F.tune_reset()
