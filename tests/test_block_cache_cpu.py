"""The cache of free device blocks over a model of the HIP runtime (native/block_cache_test.cpp): what needs
two devices, or a stream whose work is still running, without a GPU."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SOURCE = os.path.join(HERE, "native", "block_cache_test.cpp")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("block_cache") / "test")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    # host code over the runtime's C interface alone
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unused-function", "-D__HIP_PLATFORM_AMD__",
                           f"-I{rocm}/include", SOURCE, "-o", out, "-lpthread"])
    return out


@pytest.mark.parametrize("case", ["events_by_device", "unfinished_elsewhere", "other_device_is_trimmed"])
def test_block_cache(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
