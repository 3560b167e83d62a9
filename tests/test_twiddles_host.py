"""The staged twiddle tables (fsa_fft.hpp) hold, at the place each stage of a
transform reads, bit for bit the plain table's value: every supported length,
both radix families, both directions (tests/host/staged_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_staged_tables_equal_the_plain_one(tmp_path):
    exe = tmp_path / "staged_check"
    src = os.path.join(ROOT, "tests", "host", "staged_check.cpp")
    subprocess.run(["g++", "-O1", "-std=c++17", src, "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip() == "ok"
