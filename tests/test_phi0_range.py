"""phi0 of an ellipsoid ends its bisection early where a few evaluations around a Newton
estimate settle it; the result must stay that of every step.  The device header, compiled for
the host over the HIP emulation, against the oracle bit for bit, where the estimate is worst:
flat and nearly equal semi-axes, points on the surface, magnitudes far from 1."""
import os
import subprocess

import pytest

from tests.cpu_hip import emu

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "cpu_hip")
pytestmark = pytest.mark.skipif(not os.path.exists(emu.CLANG), reason="no host clang++")


# (the library's sources are compiled with and without contraction)
@pytest.mark.parametrize("contract", ["on", "off"])
def test_phi0_range_bitwise_equal_to_oracle(tmp_path, contract):
    import oracle
    lib = oracle.build(force=False)
    exe = str(tmp_path / "phi0_range_check")
    subprocess.check_call([emu.CLANG, "-std=c++20", "-O2", "-Wno-unknown-attributes",
                           "-ffp-contract=" + contract, "-I", HERE,
                           "-I", os.path.join(emu.ROOT, "include"), "-I", emu.CSRC,
                           "-x", "c++", os.path.join(HERE, "phi0_range_check.cpp"), "-x", "none",
                           lib, "-Wl,-rpath," + os.path.dirname(lib), "-o", exe])
    out = subprocess.run([exe, "400000"], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "400000 points, 0 mismatches" in out.stdout
