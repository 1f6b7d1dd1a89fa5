"""Bricks whose cells spread over more columns than are staged are fitted in two halves, against the
oracle: small balls whose layers lie in few bricks, with and without the normal factor."""
import numpy as np
import pytest

import helpers
from cpu_hip import emu
from paper_2104_00095_amd import fields, rmx, synth


def ball(at, radius=4.0, n=28, n_layers=4, spacing=None):
    """A ball of `radius` cells around cell `at` of an n^3 box, under a smooth map."""
    h = 1.0 / n
    w = synth.Workload("ball", (n, n, n), h, (0.0, 0.0, 0.0))
    if spacing is not None:
        w.spacing = tuple(h * s for s in spacing)
    x, y, z = synth.cell_centres((0, 0, 0), (n, n, n), h, (0.0, 0.0, 0.0))
    xi = np.stack(np.broadcast_arrays(x + 0.02 * np.sin(4 * y), y + 0.03 * z * x,
                                      z + 0.02 * np.cos(3 * x)))
    mid = [float(xi[a][at[2], at[1], at[0]]) for a in range(3)]
    w.solids.append(synth.Solid((0, 0, 0), (n, n, n), synth.sphere_shape(mid, radius * h),
                                n_layers, np.ascontiguousarray(xi)))
    return w


def columns(lab, layer):
    """The most columns that a brick of the layer stages: row by row from the first to the last
    within 2 of one of its cells."""
    n = lab.shape[0]
    on = np.pad(lab == layer, ((2, 10),) * 3)
    most = 0
    for b in np.ndindex((n + 7) // 8, (n + 7) // 8, (n + 7) // 8):
        t = np.zeros((16, 16, 16), bool)
        t[4:12, 4:12, 4:12] = on[tuple(slice(2 + 8 * i, 10 + 8 * i) for i in b)]
        near = np.zeros((12, 12, 12), bool)
        for d in np.ndindex(5, 5, 5):
            near |= t[d[0]:d[0] + 12, d[1]:d[1] + 12, d[2]:d[2] + 12]
        first, last = near.argmax(axis=2), 11 - near[:, :, ::-1].argmax(axis=2)
        most = max(most, int(np.where(near.any(axis=2), last - first + 1, 0).sum()))
    return most


# (the ball's middle in the middle of a brick: its first layers lie in that brick alone)
CASES = {"normals": (dict(at=(12, 12, 12)), 1), "plain": (dict(at=(11, 12, 12), radius=3.2), 3),
         "spacings": (dict(at=(12, 12, 12), spacing=(1.0, 1.3, 0.8)), 1)}


def compare(name, w, got):
    xi, lab, dec = got
    so, xo, lo, do, _ = helpers.run_oracle(w, w.solids[0])
    assert so == 0
    assert columns(lo, CASES[name][1]) > 1440   # the case is one
    assert np.array_equal(lab, lo) and np.array_equal(dec, do)
    # (the parity bar, times up to 1e3 for the conditioning of a ball of four cells)
    assert helpers.rel_err(xi, xo, lo > 0) <= 1e-9


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, 16])   # the launch chain, the persistent launch
@pytest.mark.parametrize("name", sorted(CASES))
def test_gpu_halves(name, flags):
    w = ball(**CASES[name][0])
    dw = fields.upload(w, decisions=True)
    ctx = rmx.Context(0)
    st, _ = ctx.extrapolate(dw.grid, dw.solids, rmx.options(flags=flags))
    assert st == 0
    got = (dw.xi[0].cpu().numpy(), dw.labels[0].cpu().numpy(), dw.decisions[0].cpu().numpy())
    ctx.close()
    compare(name, w, got)


@pytest.mark.parametrize("name", ["normals"])
def test_emulated_halves(name, tmp_path):
    w = ball(**CASES[name][0])
    st, outs = emu.run(w, str(tmp_path))
    assert st == 0
    compare(name, w, outs[0][:3])
