"""Where the launches of a call end, checked on the host: tests/host/check_launch_cuts.cpp is built with the plain C++ compiler
against the header that asgd_run_steps() uses (csrc/launch_cuts.h)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launches_are_the_steps_of_the_call(tmp_path):
    exe = str(tmp_path / "check_launch_cuts")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_1505_04956_amd", "csrc"), "-o", exe,
                           os.path.join(ROOT, "tests", "host", "check_launch_cuts.cpp")])
    out = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert out.returncode == 0 and out.stdout.startswith("ok "), out.stdout
