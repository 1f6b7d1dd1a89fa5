"""Time steps of batches past the 64 solids that a wave looks up at a time, against the oracle."""
import numpy as np
import pytest

from paper_2104_00095_amd import synth
from tests.helpers import StepCase, compare_step
from tests.test_gpu_step import ctx, gpu_step   # noqa: F401


def step_spheres(n):
    """n spheres of radius 2.5 cells on a lattice, in boxes of 19 to 22 cells a side: five layers
    and the predictor's three cells fit."""
    per = 6
    h = 1.0 / 22
    side = 22 * per
    w = synth.Workload("step_spheres", (side, side, 22 * ((n + per * per - 1) // (per * per))), h,
                       (0.0, 0.0, 0.0))
    for i in range(n):
        at = (22 * (i % per), 22 * (i // per % per), 22 * (i // (per * per)))
        ext = tuple(19 + (i + a) % 4 for a in range(3))
        x, y, z = synth.cell_centres(at, ext, h, (0.0, 0.0, 0.0))
        xi = np.stack(np.broadcast_arrays(x + 0.01 * np.sin(4 * y), y + 0.02 * z * x,
                                          z + 0.01 * np.cos(3 * x)))
        mid = [float(xi[a][ext[2] // 2, ext[1] // 2, ext[0] // 2]) for a in range(3)]
        w.solids.append(synth.Solid(at, ext, synth.sphere_shape(mid, 2.5 * h), 5,
                                    np.ascontiguousarray(xi)))
    return w


@pytest.mark.gpu
@pytest.mark.parametrize("n", [65, 130])
def test_gpu_step_of_many_solids(ctx, n):   # noqa: F811
    case = StepCase(step_spheres(n))
    st, got = gpu_step(ctx, case)
    assert st == 0
    expect = [(o[0], o[1], o[2], o[3], o[5]) for o in case.oracle()]
    compare_step(case, got, expect, tag=n)
