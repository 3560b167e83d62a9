"""Which schedule a small 3D grid takes: the kernels one fsa_apply enqueues, counted in
a captured graph (3 with passes B, C and D in one launch, 5 apart)."""
import ctypes

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
    ((24, 64, 48), "f64", 5), ((24, 64, 64), "f64", 3), ((12, 96, 96), "f64", 3), ((96, 16, 96), "f64", 3),
    ((12, 96, 8), "f32", 3), ((96, 8, 8), "f64", 3),
    # past the plane's size, and an axis longer than 128
    ((48, 48, 8), "f32", 5), ((8, 192, 8), "f32", 5),
])
def test_untuned_schedule(F, N, prec, want):
    plan, rho = make(F, N, prec)
    assert kernels(plan, rho) == want
