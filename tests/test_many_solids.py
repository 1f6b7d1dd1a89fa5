"""Batches around the 64 solids that a wave looks up at a time: every solid's chunks must be found,
against the oracle, at one, 64, 65 and 130 solids."""
import numpy as np
import pytest

import helpers
from paper_2104_00095_amd import fields, rmx, synth


def small_spheres(n):
    """n spheres of radius 2.5 cells on a lattice, in boxes of 9 to 12 cells a side."""
    per = 6
    h = 1.0 / 12
    side = 12 * per
    w = synth.Workload("small_spheres", (side, side, 12 * ((n + per * per - 1) // (per * per))), h,
                       (0.0, 0.0, 0.0))
    for i in range(n):
        at = [12 * (i % per), 12 * (i // per % per), 12 * (i // (per * per))]
        ext = tuple(9 + (i + a) % 4 for a in range(3))
        x, y, z = synth.cell_centres(tuple(at), ext, h, (0.0, 0.0, 0.0))
        xi = np.stack(np.broadcast_arrays(x + 0.01 * np.sin(4 * y), y + 0.02 * z * x,
                                          z + 0.01 * np.cos(3 * x)))
        mid = [float(xi[a][ext[2] // 2, ext[1] // 2, ext[0] // 2]) for a in range(3)]
        shape = synth.sphere_shape(tuple(mid), 1.6 * h)
        w.solids.append(synth.Solid(tuple(at), ext, shape, 1, np.ascontiguousarray(xi)))
    return w


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 64, 65, 130])
def test_gpu_many_solids(n):
    w = small_spheres(n)
    dw = fields.upload(w, decisions=True)
    ctx = rmx.Context(0)
    st, _ = ctx.extrapolate(dw.grid, dw.solids, rmx.options())
    assert st == 0
    for i, s in enumerate(w.solids):
        so, xo, lo, do, _ = helpers.run_oracle(w, s)
        assert so == 0, (i, so)
        assert (lo > 0).any() and (lo == 0).any(), i
        assert np.array_equal(dw.labels[i].cpu().numpy(), lo), i
        assert np.array_equal(dw.decisions[i].cpu().numpy(), do), i
        # (the parity bar of the FP64 fits)
        assert helpers.rel_err(dw.xi[i].cpu().numpy(), xo, lo > 0) <= 1e-12, i
    ctx.close()
