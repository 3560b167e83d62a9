"""Waves per SIMD that the compiler's resource report gives kernels at the edge of a
register step, compiled for the GPU with the library's own flags (no GPU needed)."""
import re
import shutil
import subprocess

import pytest

from paper_2504_19410_amd import build as B


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_rows_of_24_keep_three_waves(tmp_path):
    src = tmp_path / "k.hip"
    src.write_text('#include "fsa_internal.hpp"\n#include "fsa_passes.hpp"\nnamespace fsa {\n'
                   "template __global__ void k_c2r<float, 24, 0, JobOne<JobC2r>>(\n"
                   "    JobOne<JobC2r>, const cpx<float>*, const cpx<float>*);\n}\n")
    r = subprocess.run(["hipcc", *B.CXXFLAGS, "-Rpass-analysis=kernel-resource-usage", "-I",
                        B.CSRC, "-c", str(src), "-o", str(tmp_path / "k.o")],
                       capture_output=True, text=True, cwd=tmp_path)
    assert r.returncode == 0, r.stderr[-2000:]
    waves = [int(x) for x in re.findall(r"Occupancy \[waves/SIMD\]: (\d+)", r.stderr)]
    assert waves == [3], r.stderr[-2000:]
