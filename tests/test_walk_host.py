"""Pass C's even walk over its work items, on the CPU (tests/host/even_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_even_walk(tmp_path):
    exe = tmp_path / "even_check"
    src = os.path.join(ROOT, "tests", "host", "even_check.cpp")
    subprocess.run(["g++", "-O2", "-std=c++17", src, "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "OK" in r.stdout, r.stdout + r.stderr
