"""Addresses of the adjoint tile's loads, checked on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_adjoint_tile_loads_stay_in_the_callers_states(tmp_path):
    exe = str(tmp_path / "tile_read")
    subprocess.run(["hipcc", "--offload-host-only", "-std=c++17", "-O1",
                    "-I", os.path.join(ROOT, "paper_2309_02825_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "tile_read.hip")], check=True)
    assert subprocess.run([exe], capture_output=True, text=True, check=True).stdout == "ok\n"
