"""Host logic of the graded streaming by source cell (no GPU): compiles a
driver against the library's table builder (csrc/tables.cpp)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_cell_readers_partition_and_transpose(tmp_path):
    csrc = os.path.join(ROOT, "paper_2012_05537_amd", "csrc")
    exe = os.path.join(tmp_path, "readers_check")
    subprocess.check_call([HIPCC, "-O1", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                           "-I", os.path.join(ROOT, "include"), "-I", csrc,
                           os.path.join(ROOT, "tests", "host", "readers_check.cpp"),
                           os.path.join(csrc, "tables.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
