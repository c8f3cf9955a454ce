"""The plan code's choices, checked without a GPU: the built library against a HIP
runtime that keeps its memory on the host and records launches instead of running
them (host/fake_hip.hpp).  Each check is one function of host/plan_paths_driver.cpp."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2609_12476_amd")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not shutil.which("g++") or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("no host compiler or no HIP headers")
    if not os.path.exists(os.path.join(PKG, "libnufft_resample.so")):
        pytest.skip("the library is not built")
    exe = tmp_path_factory.mktemp("plan_paths") / "driver"
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-w", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(PKG, "csrc"), "-isystem", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "host", "plan_paths_driver.cpp"), "-rdynamic", "-o", str(exe),
                    "-L", PKG, "-lnufft_resample", f"-Wl,-rpath,{PKG}:/opt/rocm/lib", "-Wl,--allow-shlib-undefined"],
                   check=True)
    return str(exe)


@pytest.mark.parametrize("check", ["strict", "fallback", "full_lds", "large_launches", "tuner", "groups", "copies",
                                   "records", "plan_time", "worth"])
def test_plan_paths(driver, check):
    r = subprocess.run([driver, check], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-2000:]
