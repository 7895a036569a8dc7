"""How the getters' results reach the host (stage.h, compiled for the host with its HIP calls
replaced): packed by one launch on the arrays' own device, by plain copies where another
device is current, without pinned memory, and above the stage's size."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_results_reach_the_host(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")):
        pytest.skip("no g++ or HIP headers")
    exe = str(tmp_path / "stage_host")
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-w",
                    os.path.join(HERE, "stage_host.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout
    rows = {r.split()[0]: r.split()[1:] for r in out.splitlines()}
    assert rows["same"] == ["1", "0", "1", "right"]
    assert rows["second"] == ["1", "0", "1", "right"]
    for name in ("other", "unpinned", "large"):
        assert rows[name] == ["0", "2", "1", "right"], name
