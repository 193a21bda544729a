"""The matrix of the first pass of 8-bit records holds no fewer bits than FP32
(tests/cpp/test_matrix.cpp: host code of the library's header, on the CPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1509_00186_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")
def test_matrix_fragments(tmp_path):
    exe = str(tmp_path / "test_matrix")
    subprocess.run([HIPCC, "-std=c++17", "-O1", "--offload-host-only", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), "-x", "hip",
                    os.path.join(ROOT, "tests", "cpp", "test_matrix.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "all passed" in r.stdout
