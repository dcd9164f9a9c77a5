"""No kernel reads a value that nothing has set, by the compiler's static
analyser over the device code (hipcc's clang; nothing is built or run)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_27210_amd", "csrc")
CLANG = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")


@pytest.mark.parametrize("source", ["fv_kernels.hip", "fv_calib.hip"])
def test_no_uninitialised_read(source, tmp_path):
    if not os.path.exists(CLANG):
        pytest.skip("no ROCm clang")
    # 20,000 states per function: 10 s, and the whole of what a default run
    # (225,000 states, 60 s) reports
    res = subprocess.run(
        [CLANG, "--analyze", "-x", "hip", "--cuda-device-only", "--offload-arch=gfx950", "-nogpulib",
         "-std=c++17", "-I", os.path.join(ROOT, "include"), "-Xclang", "-analyzer-checker=core", "-Xclang",
         "-analyzer-output=text", "-Xclang", "-analyzer-config", "-Xclang", "max-nodes=20000",
         os.path.join(CSRC, source)], cwd=str(tmp_path), capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    found = [line for line in res.stderr.splitlines() if "[core." in line]
    assert not found, found
