"""The LDS layout of the step kernels with fp16-split operands, checked on the host: tests/host/check_split_plan.cpp is built with the
plain C++ compiler against the header that the launcher uses (csrc/split_plan.h)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "check_split_plan")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_1505_04956_amd", "csrc"), "-o", exe,
                           os.path.join(ROOT, "tests", "host", "check_split_plan.cpp")])
    return exe


# every k and one mini-batch size in three of the usual ones, row lengths around the chunks of 16 columns, few and many workers
@pytest.mark.parametrize("d", [1, 3, 7, 8, 12, 15, 16, 17, 32, 33, 48, 60, 64, 65, 100, 128, 129, 384, 8192])
@pytest.mark.parametrize("W", [1, 192, 256, 300])
def test_layout_fits_a_compute_unit(checker, d, W):
    out = subprocess.run([checker, str(d), str(W)], stdout=subprocess.PIPE, text=True)
    assert out.returncode == 0 and out.stdout.startswith("ok "), out.stdout
    if d <= 64 and W == 192:
        assert int(out.stdout.split()[3]) > 1000


# rows of more than 128 columns, workers that do and do not divide the compute units evenly: the cut of the mini-batches
@pytest.mark.parametrize("W", [64, 100, 129, 150, 190, 257, 400, 600])
def test_long_rows_fill_the_device(checker, W):
    out = subprocess.run([checker, "384", str(W)], stdout=subprocess.PIPE, text=True)
    assert out.returncode == 0 and out.stdout.startswith("ok "), out.stdout
