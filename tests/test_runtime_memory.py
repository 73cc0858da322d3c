"""Device memory of the host runtime (CPU only): runtime.cpp over a HIP runtime and launchers on the
host (tests/native/fake_hip.h), which check every range that a launch would read or write against
the live allocations, under budgets and device limits from too small to ample."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1912_06636_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")):
        pytest.skip("needs g++ and the HIP headers")
    exe = str(tmp_path_factory.mktemp("runtime") / "runtime_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__",
                    "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-isystem", os.path.join(ROCM, "include"),
                    os.path.join(ROOT, "tests", "native", "runtime_check.cpp"),
                    os.path.join(CSRC, "runtime.cpp"), os.path.join(CSRC, "plan.cpp"), "-o", exe, "-lpthread"], check=True)
    return exe


@pytest.mark.parametrize("scenario", ["scratch", "arrays", "regroup"])
def test_launches_stay_in_live_memory(program, scenario):
    r = subprocess.run([program, scenario], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and scenario + ": all ok" in r.stdout, r.stdout + r.stderr[-4000:]
