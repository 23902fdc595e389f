"""Host logic of the streaming launches (no GPU): compiles a driver against the
library's sources and runs one check of it per test."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    csrc = os.path.join(ROOT, "paper_2012_05537_amd", "csrc")
    exe = os.path.join(tmp_path_factory.mktemp("launch"), "launch_check")
    subprocess.check_call([HIPCC, "-O1", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                           "-I", os.path.join(ROOT, "include"), "-I", csrc,
                           os.path.join(ROOT, "tests", "host", "launch_check.cpp"),
                           os.path.join(csrc, "tables.cpp"), os.path.join(csrc, "tables_mapped.cpp"),
                           os.path.join(csrc, "layouts.cpp"), "-o", exe])
    return exe


@pytest.mark.parametrize("check", ["run_grids", "layouts", "lds_of_block", "nontemporal_rows", "short_runs"])
def test_launch(driver, check):
    out = subprocess.run([driver, check], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
