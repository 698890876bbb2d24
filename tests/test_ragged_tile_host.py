"""Host check of the LDS tiles of ragged calls on frequency nodes (ragged_tile_check.cpp)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.join(os.path.dirname(__file__), "..")
CSRC = os.path.join(ROOT, "paper_1904_02863_amd", "csrc")


def test_ragged_tiles(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not installed")
    with open(os.path.join(CSRC, "gw_phasor_table.h")) as fh:
        entries = int(re.search(r"#define GW_PHTAB_N (\d+)", fh.read()).group(1))
    exe = tmp_path / "ragged_tile_check"
    subprocess.run([hipcc, "-std=c++17", "-O1", f"-DPHASOR_TABLE_BYTES={16 * entries}", "-I",
                    os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "ragged_tile_check.cpp"),
                    "-o", str(exe)], check=True, capture_output=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
    assert out.stdout.startswith("ok ")
