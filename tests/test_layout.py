"""Rules of the layout header that kernels and host code share, compiled for
the host (no GPU)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_layout_rules(tmp_path):
    exe = str(tmp_path / "layout_test")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-fsanitize=undefined", "-D__HIP_PLATFORM_AMD__",
                    "-isystem", os.path.join(ROCM, "include"), "-o", exe, os.path.join(HERE, "cpp", "layout_test.cpp")],
                   check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=120)
    assert "layout ok" in out.stdout
