"""The largest term that fixed-point sums may hold where column maxima are formed of a part of the samples, checked on the host:
tests/host/check_term_limit.cpp is built with the plain C++ compiler against the kernel's header (csrc/fixed_point_sums.h)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_limit_of_a_term(tmp_path):
    exe = str(tmp_path / "check_term_limit")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_1505_04956_amd", "csrc"), "-o", exe,
                           os.path.join(ROOT, "tests", "host", "check_term_limit.cpp")])
    for b in (1, 2, 63, 255, 256, 300, 500, 511, 512, 513, 1000, 4096, 65535, 1 << 20):
        out = subprocess.run([exe, str(b)], stdout=subprocess.PIPE, text=True)
        assert out.returncode == 0 and out.stdout.startswith("ok "), out.stdout
