"""The host-side plans of the kernels (LDS, strips, tiles) over every size the library accepts.  They are
plain C++ without HIP, so the checks of tests/plan_check.cpp run without a GPU: a plan that asks for more
LDS than a compute unit has, or a tile that misses pixels, shows here and not as a failing launch."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_plans_of_all_sizes(tmp_path):
    exe = str(tmp_path / "plan_check")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2304_04237_amd", "csrc"),
                           os.path.join(ROOT, "tests", "plan_check.cpp"), "-o", exe])
    run = subprocess.run([exe], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
