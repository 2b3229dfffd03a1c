"""The GPU compressor's host code on the CPU (encode_host_driver.hip): its
device memory where that is short, and its state after calls that failed."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which(HIPCC) is None:
        pytest.skip("needs hipcc")
    d = tmp_path_factory.mktemp("encode_host")
    obj, exe = str(d / "driver.o"), str(d / "driver")
    subprocess.run([HIPCC, "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-pthread", "-c",
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "encode_host_driver.hip"),
                    "-o", obj], check=True)
    # no GPU code is linked, and none of the HIP runtime
    subprocess.run([os.path.join(os.path.dirname(os.path.realpath(HIPCC)), "..", "llvm", "bin", "clang++"), obj,
                    "-pthread", "-Wl,--unresolved-symbols=ignore-all", "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("scenario", ["plain", "smaller arenas", "small after too large", "every failure",
                                      "batches"])
def test_host_code_of_the_gpu_compressor(driver, scenario):
    r = subprocess.run([driver, scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
