"""The rule that chooses between the 3D step kernels (csrc/fd_plan.hpp), on
the host: sizes timed with both kernels take the faster one."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_sizes_take_the_faster_kernel(tmp_path):
    exe = str(tmp_path / "plan_checks")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-fsanitize=undefined",
                    "-fno-sanitize-recover=all", os.path.join(ROOT, "tests", "native", "plan_checks.cpp"), "-o", exe],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "plan checks passed" in r.stdout, r.stdout + r.stderr
