"""The plans of the kernels in the momentum transform (csrc/kspace_plan.h), checked on the
host over many shapes: what each wave and lane takes, and that it stays inside its buffers."""
import os
import subprocess

import pytest

from paper_1912_10024_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_check")
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-I" + os.path.join(build.ROOT, "include"),
                    "-I" + os.path.join(build.HERE, "csrc"), os.path.join(HERE, "plan_check.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("check", ["first_task", "corr_window", "corr_search_time", "corr_support", "launch_parts"])
def test_plan(checker, check):
    res = subprocess.run([checker, check], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout
