"""The consumers' fill: more units than one launch takes at once, regions of many units that wrap
around a periodic end, and more solids than a wave looks up at a time, against the oracle."""
import os
import subprocess

import numpy as np
import pytest

from paper_2104_00095_amd import rmx, synth
from tests.cpu_hip import emu
from tests.helpers import BlurCase, compare_blur
from tests.test_blur_tiles import scattered_blur
from tests.test_gpu_blur import ctx, gpu_blur   # noqa: F401
from tests.test_many_solids import small_spheres

# Boxes that span whole planes of 40 x 36 from z = 9, 17 and 23 on: runs that end at the last
# plane, straddle it and start behind it, in up to five units each.  With the rows of the last
# two boxes 1400 units of the stress, past the 1024 that the emulated device's grid takes at once.
PERIODIC = ((40, 36, 24), (1, 1, 1),
            [((3, 5, 9), (40, 36, 24)), ((0, 0, 17), (40, 36, 12)), ((39, 1, 23), (40, 36, 9)),
             ((30, 30, 20), (20, 11, 9)), ((2, 3, 1), (30, 33, 20))])


def periodic_case():
    return scattered_blur(PERIODIC, ("sphere", "ellipsoid"), 31)


def test_grid_of_the_fill(tmp_path):
    """The grid stays below the launch limit whatever the number of units (2^26 units, one wave
    each, are past it)."""
    here = os.path.join(os.path.dirname(os.path.abspath(__file__)), "cpu_hip")
    exe = str(tmp_path / "fill_blocks_check")
    subprocess.check_call([emu.CLANG, "-std=c++20", "-O1", "-Wno-unknown-attributes", "-I", here,
                           "-I", emu.CSRC, "-x", "c++",
                           os.path.join(here, "fill_blocks_check.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr


def test_emulated_periodic_planes(tmp_path):
    c = periodic_case()
    st, H, phis, taus = emu.run_blur(c.w, str(tmp_path), c.xi, c.labels, c.eps, c.G, c.H_init,
                                     c.phi_init, c.tau_init)
    assert st == 0
    compare_blur(c, (H, phis, taus), c.oracle())


@pytest.mark.gpu
def test_gpu_periodic_planes(ctx):   # noqa: F811
    case = periodic_case()
    compare_blur(case, gpu_blur(ctx, case), case.oracle())


@pytest.mark.gpu
@pytest.mark.parametrize("n", [65, 130])
def test_gpu_many_solids(ctx, n):   # noqa: F811
    case = BlurCase(small_spheres(n), eps_cells=1.0)
    compare_blur(case, gpu_blur(ctx, case), case.oracle(), tag=n)


@pytest.mark.gpu
def test_gpu_more_units_than_a_launch(ctx):   # noqa: F811
    """460 boxes of 1 x 1 x 8184 cells on one place: 147 318 units of the stress each, more than
    2^26 in all.  None is covered, so every face of the boxes gets zero and no other is written."""
    import torch
    n, length = 460, 8184
    h = 1.0 / 16
    grid = rmx.grid((3, 3, length), h, (0.0, 0.0, 0.0))
    xi = torch.zeros((3, length, 1, 1), dtype=torch.float64, device="cuda")
    lab = torch.full((length, 1, 1), -1, dtype=torch.int8, device="cuda")
    s = synth.sphere_shape((0.0, 0.0, 0.0), 0.1)
    sols = [rmx.solid((1, 1, 0), (1, 1, length), rmx.shape(s.kind, s.centre, s.semi, s.rot), 1, xi,
                      lab) for _ in range(n)]
    units = 6 * (length + length + length + 1)
    assert n * units >= 1 << 26
    taus = [torch.full((6, length + (a == 2), 3 + (a == 1), 3 + (a == 0)), 7.0,
                       dtype=torch.float64, device="cuda") for a in range(3)]
    ctx.solid_stress(grid, sols, h, [1.0] * n, taus)
    torch.cuda.synchronize()
    for a in range(3):
        got = taus[a].cpu().numpy()
        want = np.full(got.shape, 7.0)
        want[:, :, 1:2 + (a == 1), 1:2 + (a == 0)] = 0.0
        assert np.array_equal(got, want), a
