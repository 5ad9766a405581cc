"""What the host code allocates, launches, captures and replays, checked without
a GPU: csrc/pn_api.hip compiled for the host alone, linked with the HIP runtime
stand-in of host_calls.cpp (which records calls and runs no kernel)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    gxx = shutil.which("g++")
    if not os.path.exists(hipcc) or gxx is None:
        pytest.skip("hipcc or g++ not available")
    tmp = tmp_path_factory.mktemp("host_calls")
    obj, exe = str(tmp / "host_calls.o"), str(tmp / "host_calls")
    subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-g",
                    "-std=c++17", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1801_07986_amd", "csrc"), "-c",
                    os.path.join(ROOT, "tests", "host_calls.cpp"), "-o", obj], check=True)
    # the device code (__hip_fatbin_*) is not there and not needed
    subprocess.run([gxx, obj, "-o", exe, "-no-pie", "-Wl,--unresolved-symbols=ignore-all",
                    "-lpthread"], check=True)
    return exe


@pytest.mark.parametrize("check", ["stage_shape", "noalloc", "graph_count", "caller_captures",
                                   "ensemble_epilogues"])
def test_host_calls(driver, check):
    env = {k: v for k, v in os.environ.items() if not k.startswith("PN_")}
    run = subprocess.run([driver, check], capture_output=True, text=True, timeout=120, env=env)
    assert run.returncode == 0, run.stderr[-2000:]
    assert f"{check} ok" in run.stdout
