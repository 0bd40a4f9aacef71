"""The bounds of the SCF workspace that a context keeps, on the CPU (no GPU, no HIP runtime)."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_workspace_is_bounded_and_given_up(tmp_path):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    exe = tmp_path / "scf_workspace_check"
    src = os.path.join(ROOT, "tests", "native", "scf_workspace_check.cpp")
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__",
                          "-I" + os.path.join(rocm, "include"), "-o", str(exe), src],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0 and run.stdout.strip() == "OK", run.stdout
