"""What smat_spmm enqueues when several threads, the per-thread stream or a graph capture share a handle: host code alone, built
here against launchers that write down their order (host/recorded_calls.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2408_11551_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(not shutil.which("g++"), reason="needs g++")
def test_areas_are_never_shared_by_launches_that_may_overlap(tmp_path):
    exe = str(tmp_path / "recorded_calls")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(ROCM, "include"),
                    os.path.join(ROOT, "tests", "host", "recorded_calls.cpp"),
                    *(os.path.join(CSRC, f) for f in ("api.cpp", "preprocess.cpp", "workers.cpp")), "-o", exe], check=True)
    out = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=100)
    assert out.returncode == 0 and out.stdout.strip() == "OK", out.stdout
