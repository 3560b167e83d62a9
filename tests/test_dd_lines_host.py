"""Lines per workgroup of the double-double transforms, on the CPU
(tests/host/dd_lines_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_small_launches_take_a_wave_per_workgroup(tmp_path):
    exe = tmp_path / "dd_lines_check"
    src = os.path.join(ROOT, "tests", "host", "dd_lines_check.cpp")
    subprocess.run(["g++", "-O2", "-std=c++17", src, "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
