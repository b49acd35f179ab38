"""The block cache behind the default allocator over a model of the HIP calls
it makes (devmem_model.cpp): orders between streams, captures and failures that
no GPU run shows reliably, or that may not be run there."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("devmem") / "model")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-x", "c++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", f"{rocm}/include",
                    "-I", os.path.join(ROOT, "paper_2506_01576_amd", "csrc"), "-pthread", "-o", exe,
                    os.path.join(ROOT, "tests", "devmem_model.cpp")], check=True)
    return exe


@pytest.mark.parametrize("scenario", ["order", "capture_elsewhere", "failed_wait", "memory_short", "trim",
                                      "other_device", "null_left_idle"])
def test_devmem_model(model, scenario):
    r = subprocess.run([model, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
