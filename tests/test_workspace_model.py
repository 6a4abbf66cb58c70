"""The library's workspace code (kept blocks of the null stream) built for the host against a model
of the HIP runtime: bounds, reuse, a release that returns every kept block, kept blocks that make
room for any stream's workspace, and several host threads on the null stream at once."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2310_01889_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_workspace_against_model(tmp_path):
    exe = str(tmp_path / "workspace_model")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"),
                    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-x", "c++", os.path.join(CSRC, "workspace.hip"),
                    os.path.join(HERE, "fake_hip_workspace.cpp"), "-o", exe, "-lpthread"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
