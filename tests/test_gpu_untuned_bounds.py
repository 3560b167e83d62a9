"""The bound under which the untuned real passes, FP64 at 768, take variant 3: a workgroup
(4 rows) on every CU of this device at most."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_real_passes_of_768_follow_the_cus():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_19410_amd import fsa as F
    F.tune_reset()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for p in ("r2c", "c2r"):
        assert F.tune_get("f64", p, 768, 4 * cus)[0] == 3
        assert F.tune_get("f64", p, 768, 4 * cus + 1)[0] == 0
        assert F.tune_get("f64", p, 768, 1 << 30)[0] == 0
