"""The slice scheduler (launches in flight, yields, decode and prefill taking turns) and the uploads against a model of the GPU's
streams: native/scheduler_check.cpp, linked with the library as it is built, in the place of the HIP runtime."""
import os
import subprocess

import pytest

import paper_2604_07874_amd.build as B   # not a `from` import, which would load the library (before torch has loaded its HIP runtime)

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(B.LIB):
        B.build(verbose=False)
    out = str(tmp_path_factory.mktemp("native") / "scheduler_check")
    cmd = [B.hipcc_path(), "-x", "hip", "--offload-host-only", "-O1", "-g", "-std=c++17", "-rdynamic",
           "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC, os.path.join(HERE, "native", "scheduler_check.cpp"),
           "-o", out, "-L", B.HERE, "-lvalvekv", f"-Wl,-rpath,{B.HERE}", "-pthread"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return out


@pytest.mark.parametrize("check", ["bound", "lower_limit", "taking_turns", "yield_between", "late_start", "failed_stream",
                                   "long_waits", "recorded", "failed_launch", "failed_copy",
                                   "overlap_rule"])
def test_scheduler(program, check):
    try:
        res = subprocess.run([program, check], capture_output=True, text=True, timeout=30)
    except subprocess.TimeoutExpired:
        pytest.fail(f"{check}: the scheduler waits for something that does not come")
    assert res.returncode == 0, res.stdout + res.stderr
