"""The workspace layouts against the kernels that read them, on the host, over the sizes at which a rule of the layout or of a
dispatch changes: no GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")
def test_layouts_fit_their_kernels(tmp_path):
    exe = tmp_path / "layout_check"
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-w", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-mllvm", "-amdgpu-mfma-vgpr-form=1", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2009_13977_amd", "csrc"), "-o", str(exe), os.path.join(ROOT, "tests", "layout_check.hip")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:]
    assert " 0 failures" in r.stdout
