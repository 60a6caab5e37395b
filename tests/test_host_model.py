"""The library's host code on a model of the HIP runtime (tests/c/host_model.cpp), built with
g++: allocations, copies and pointers that no device is needed for, or that a device must not
be given wrong."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_host_code_on_a_model_of_the_runtime(tmp_path):
    csrc = os.path.join(ROOT, "paper_1607_03062_amd", "csrc")
    include = [os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), os.path.join(ROOT, "include"), csrc]
    exe = tmp_path / "host_model"
    subprocess.run(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-Wall", "-Wno-unused-result",
                    "-D__HIP_PLATFORM_AMD__", *["-I" + d for d in include],
                    os.path.join(ROOT, "tests", "c", "host_model.cpp"), os.path.join(csrc, "pd_api.cpp"),
                    os.path.join(csrc, "field.cpp"), "-o", str(exe), "-lpthread"], check=True, capture_output=True,
                   text=True)
    env = dict(os.environ)
    env.pop("PD_FAULT", None)
    r = subprocess.run([str(exe)], capture_output=True, text=True, env=env, timeout=120)
    assert r.returncode == 0 and "host model ok" in r.stdout, r.stdout[-4000:] + r.stderr[-2000:]
