"""The layer fits' staging at its edges, against the oracle: label rows read near the ends of
a box's arrays and across unaligned rows, bricks cut by the box, and bricks whose cells spread
over more columns than are staged (gathered from global memory instead)."""
import numpy as np
import pytest

import helpers
from cpu_hip import emu
from paper_2104_00095_amd import fields, rmx, synth

# Boxes whose last rows end inside a 16-byte label window, with rows of every alignment, and
# boxes with less than 16 cells (read byte by byte).
EXTENTS = [(13, 9, 8), (8, 8, 9), (17, 5, 11), (19, 16, 3), (3, 5, 1), (5, 3, 1), (16, 1, 1)]


def scattered(ext, share, seed, n_layers=2):
    """Random interior cells of a smooth map, every other cell undefined."""
    rng = np.random.default_rng(seed)
    n0, n1, n2 = ext
    mask = rng.random((n2, n1, n0)) < share
    mask[n2 // 2, n1 // 2, n0 // 2] = True
    h = 1.0 / max(ext)
    x, y, z = synth.cell_centres((0, 0, 0), ext, h, (0.0, 0.0, 0.0))
    xi = np.stack(np.broadcast_arrays(x + 0.02 * np.sin(5 * y), y + 0.03 * z * x,
                                      z + 0.02 * np.cos(4 * x)))
    xi = np.where(mask, xi, np.nan)
    w = synth.Workload("scattered", ext, h, (0.0, 0.0, 0.0))
    w.solids.append(synth.Solid((0, 0, 0), ext, synth.sphere_shape((0.5, 0.5, 0.5), 10.0),
                                n_layers, np.ascontiguousarray(xi)))
    return w


def compare(w, got, precision, tag):
    xi, lab, dec = got
    so, xo, lo, do, _ = helpers.run_oracle(w, w.solids[0])
    assert so == 0, (tag, so)
    assert np.array_equal(lab, lo), tag
    assert np.array_equal(dec, do), tag
    band = lo > 0
    # scattered data condition the 4 x 4 systems worse than a smooth surface's: condition
    # numbers up to about 1e4 over the parity bars' 1e-12 and 1e-5 / 10
    tol = 1e-3 if precision == rmx.FP32_ACCUM else 1e-9
    assert helpers.rel_err(xi, xo, band) <= tol, tag


CASES = [(e, 0.25, i) for i, e in enumerate(EXTENTS)] + [((24, 24, 24), 0.04, 50)]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [rmx.FP64, rmx.FP32_ACCUM])
@pytest.mark.parametrize("ext,share,seed", CASES)
def test_gpu_edges(ext, share, seed, precision):
    w = scattered(ext, share, seed)
    dw = fields.upload(w, decisions=True)
    ctx = rmx.Context(0)
    st, _ = ctx.extrapolate(dw.grid, dw.solids, rmx.options(precision=precision))
    assert st == 0
    got = (dw.xi[0].cpu().numpy(), dw.labels[0].cpu().numpy(), dw.decisions[0].cpu().numpy())
    ctx.close()
    compare(w, got, precision, (ext, precision))


@pytest.mark.parametrize("ext,share,seed", [CASES[0], CASES[2], CASES[4], CASES[6],
                                            ((12, 12, 12), 0.04, 51)])
def test_emulated_edges(ext, share, seed, tmp_path):
    w = scattered(ext, share, seed)
    st, outs = emu.run(w, str(tmp_path))
    assert st == 0
    compare(w, outs[0][:3], rmx.FP64, ext)
