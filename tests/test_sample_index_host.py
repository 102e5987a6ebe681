"""The elements that the column maxima over a part of the samples look at, checked on the host: tests/host/check_sample_index.cpp is
built with the plain C++ compiler against the header that the kernel uses (csrc/sample_index.h)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "check_sample_index")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_1505_04956_amd", "csrc"), "-o", exe,
                           os.path.join(ROOT, "tests", "host", "check_sample_index.cpp")])
    return exe


# the row lengths with a streaming kernel and their fewest rows: up to two sweeps of a workgroup and a few pieces, row by row; then
# the first sizes of which a part is taken, and a larger one
@pytest.mark.parametrize("k,d", [(10, 10), (4, 4), (8, 8), (8, 16), (16, 8), (16, 12)])
def test_elements_lie_inside_the_samples(checker, k, d):
    first_part = 8191 * 16 * (256 - 256 % d) // d
    for lo, hi in ((k, 2 * 256 // d + 1), (3 * 4096 // d, 3 * 4096 // d + 40), (first_part - 1, first_part + 1), (5_000_001, 5_000_001)):
        out = subprocess.run([checker, str(d), str(lo), str(hi)], stdout=subprocess.PIPE, text=True)
        assert out.returncode == 0 and out.stdout.startswith("ok "), out.stdout
