"""The blur-zone consumers at the edges of their tiles, against the oracle: scattered labels,
several solids over one face (sums of weights above 1), boxes thinner than a tile, boxes that
span whole planes of the grid (filled as runs), partial tiles, and boxes across or around
periodic ends."""
import numpy as np
import pytest

from paper_2104_00095_amd import synth
from tests.helpers import BlurCase, compare_blur
from tests.test_gpu_blur import ctx, gpu_blur   # noqa: F401

WALLED = ((21, 13, 18), (0, 0, 0),
          [((0, 0, 0), (21, 13, 18)), ((3, 2, 4), (5, 3, 2)), ((0, 5, 0), (21, 8, 9)),
           ((7, 0, 7), (14, 13, 4)), ((20, 12, 17), (1, 1, 1))])
WRAPPED = ((16, 12, 9), (1, 1, 1),
           [((5, 7, 3), (16, 12, 9)), ((14, 10, 7), (6, 5, 4)), ((0, 0, 8), (16, 12, 3))])
MIXED = ((9, 17, 16), (0, 1, 0),
         [((0, 11, 0), (9, 17, 16)), ((1, 16, 2), (8, 3, 9)), ((2, 0, 5), (3, 17, 8))])


def scattered_blur(layout, kinds, seed):
    """Smooth maps and scattered labels on the layout's boxes, a quarter of the cells outside
    0..L, about half of the rest within eps of the surfaces."""
    grid_n, periodic, boxes = layout
    rng = np.random.default_rng(seed)
    h = 1.0 / 16
    w = synth.Workload("scattered_blur", grid_n, h, (0.0, 0.0, 0.0))
    w.periodic = periodic
    c = BlurCase.__new__(BlurCase)
    c.w, c.eps, c.xi, c.labels = w, 2.0 * h, [], []
    for i, (lo, ext) in enumerate(boxes):
        x, y, z = synth.cell_centres(lo, ext, h, (0.0, 0.0, 0.0))
        centre = [(lo[a] + 0.5 * ext[a]) * h for a in range(3)]
        if kinds[i % len(kinds)] == "sphere":
            shape = synth.sphere_shape(tuple(centre), 0.3)
        else:
            shape = synth.ellipsoid_shape(tuple(centre), (0.35, 0.22, 0.28),
                                          synth.random_rotation(rng))
        xi = np.stack(np.broadcast_arrays(x + 0.02 * np.sin(5 * y), y + 0.03 * z * x,
                                          z + 0.02 * np.cos(4 * x)))
        lab = rng.integers(0, 3, size=xi.shape[1:])
        out = rng.random(lab.shape) < 0.25
        lab = np.where(out, rng.choice([-1, 3, 7], size=lab.shape), lab).astype(np.int8)
        if ext[0] * ext[1] * ext[2] < 64:
            lab[...] = 0
        w.solids.append(synth.Solid(lo, ext, shape, 2, np.ascontiguousarray(xi)))
        c.xi.append(np.ascontiguousarray(xi))
        c.labels.append(np.ascontiguousarray(lab))
    c.G = list(rng.uniform(0.5, 3.0, size=len(boxes)))
    n0, n1, n2 = grid_n
    c.H_init = np.full((n2, n1, n0), 5.0)
    c.phi_init = [np.full(x.shape[1:], -6.0) for x in c.xi]
    c.tau_init = [np.full((6, n2 + (a == 2 and not periodic[2]), n1 + (a == 1 and not periodic[1]),
                           n0 + (a == 0 and not periodic[0])), 7.0) for a in range(3)]
    return c


CASES = {"walled": (WALLED, ("ellipsoid",), 1), "wrapped": (WRAPPED, ("ellipsoid",), 2),
         "mixed": (MIXED, ("sphere", "ellipsoid"), 3),
         "spheres": (WALLED, ("sphere",), 4), "wrapped_spheres": (WRAPPED, ("sphere",), 5)}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
def test_gpu_tiles(ctx, name):   # noqa: F811
    case = scattered_blur(*CASES[name])
    compare_blur(case, gpu_blur(ctx, case), case.oracle(), tag=name)


@pytest.mark.parametrize("name", ["walled", "wrapped", "mixed", "wrapped_spheres"])
def test_emulated_tiles(name, tmp_path):
    from tests.cpu_hip import emu
    c = scattered_blur(*CASES[name])
    st, H, phis, taus = emu.run_blur(c.w, str(tmp_path), c.xi, c.labels, c.eps, c.G, c.H_init,
                                     c.phi_init, c.tau_init)
    assert st == 0
    compare_blur(c, (H, phis, taus), c.oracle(), tag=name)
