"""Host checks of the frequency nodes: the geometry of gw_nodes.h
(tests/node_check.cpp, built with hipcc and run on the CPU) and the
interpolation weights (gw_resample_weights.h is what gen_resample.py writes;
evaluated in double as the kernels do, they recover every band-limited phasor
to 5e-16, and clearly not one well outside the band)."""
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.join(os.path.dirname(__file__), "..")
CSRC = os.path.join(ROOT, "paper_1904_02863_amd", "csrc")


def test_node_geometry(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not installed")
    exe = tmp_path / "node_check"
    subprocess.run([hipcc, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "node_check.cpp"), "-o", str(exe)], check=True, capture_output=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
    assert out.stdout.startswith("ok ")


@pytest.fixture(scope="module")
def gen():
    sys.path.insert(0, CSRC)
    try:
        import gen_resample
    finally:
        sys.path.remove(CSRC)
    return gen_resample


def test_weights_header_and_error(gen):
    coef = gen.polynomials()
    with open(os.path.join(CSRC, "gw_resample_weights.h")) as fh:
        assert fh.read() == gen.header(coef)
    worst, l1 = gen.band_error(coef)
    assert worst < 5e-16 and l1 < 2.1
    assert gen.band_error(coef, nu_max=0.3)[0] > 1e-9
    # mirrored points have mirrored weights (up to rounding)
    x = np.linspace(0.0, 1.0, 11)
    assert np.abs(gen.evaluate(coef, x) - gen.evaluate(coef, 1.0 - x)[:, ::-1]).max() < 1e-15
