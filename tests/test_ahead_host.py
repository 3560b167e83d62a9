"""The transform with each stage's twiddles loaded ahead of its exchange, emulated thread
by thread on the CPU (tests/host/ahead_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_length_family_and_direction(tmp_path):
    exe = tmp_path / "ahead_check"
    src = os.path.join(ROOT, "tests", "host", "ahead_check.cpp")
    subprocess.run(["g++", "-O2", "-std=c++17", src, "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
