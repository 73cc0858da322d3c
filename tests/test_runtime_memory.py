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


def _build(directory, sanitizers):
    if shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")):
        pytest.skip("needs g++ and the HIP headers")
    exe = str(directory / "runtime_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__"] + sanitizers + [
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-isystem", os.path.join(ROCM, "include"),
                    os.path.join(ROOT, "tests", "native", "runtime_check.cpp"),
                    os.path.join(CSRC, "runtime.cpp"), os.path.join(CSRC, "plan.cpp"), "-o", exe, "-lpthread"], check=True)
    return exe


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    return _build(tmp_path_factory.mktemp("runtime"), ["-fsanitize=undefined", "-fno-sanitize-recover=all"])


@pytest.mark.parametrize("scenario", ["scratch", "arrays", "regroup", "budget", "serve"])
def test_launches_stay_in_live_memory(program, scenario):
    r = subprocess.run([program, scenario], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and scenario + ": all ok" in r.stdout, r.stdout + r.stderr[-4000:]


def test_cached_choices_of_other_kernels_are_not_taken(program, tmp_path):
    r = subprocess.run([program, "tune", str(tmp_path / "tune.json")], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "tune: all ok" in r.stdout, r.stdout + r.stderr[-4000:]


def test_clusters_given_back_beside_a_run(tmp_path):
    """The same beside another thread's launches, under ThreadSanitizer."""
    r = subprocess.run([_build(tmp_path, ["-fsanitize=thread"]), "serve"], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, TSAN_OPTIONS="halt_on_error=1"))
    if "unexpected memory mapping" in r.stderr:
        pytest.skip("ThreadSanitizer runtime does not support this kernel's memory layout")
    assert r.returncode == 0 and "serve: all ok" in r.stdout, r.stdout + r.stderr[-4000:]
