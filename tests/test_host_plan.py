"""The host-side choices of the score calls (sp_score_plan.hpp), compiled into a driver of their own: packing against its
definition on random batches, what holds for every plan, and what planning costs the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_driver")
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2603_02631_amd", "csrc"), os.path.join(ROOT, "tests", "host", "plan_driver.cpp"), "-o", exe]
    build = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert build.returncode == 0, build.stdout[-4000:]
    return exe


@pytest.mark.parametrize("what", ["packing", "plans", "ranges", "even", "whole", "cost"])
def test_plans_of_score_calls(driver, what):
    run = subprocess.run([driver, what], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert run.returncode == 0, run.stdout[-4000:]
    assert "all checks passed" in run.stdout
