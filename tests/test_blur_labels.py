"""Labels that the consumers get from their caller: a solid covers the cells it labels 0..L and
no others, so every negative label and every label above L leaves its cell out, against the
oracle (whose test is the signed comparison)."""
import numpy as np
import pytest

from tests.helpers import compare_blur
from tests.test_blur_tiles import MIXED, WALLED, WRAPPED, scattered_blur
from tests.test_gpu_blur import ctx, gpu_blur   # noqa: F401

# (the ends of the signed byte, and the negative ones whose low bits read as a layer)
OUTSIDE = np.array([-128, -127, -126, -113, -112, -2, -1, 3, 16, 17, 127], dtype=np.int8)

CASES = {"walled": (WALLED, ("ellipsoid",), 11), "wrapped": (WRAPPED, ("sphere",), 12),
         "mixed": (MIXED, ("sphere", "ellipsoid"), 13)}


def outside_labels(name):
    """The scattered labels with their outside cells on OUTSIDE and undefined maps there."""
    layout, kinds, seed = CASES[name]
    c = scattered_blur(layout, kinds, seed)
    rng = np.random.default_rng(seed)
    for xi, lab in zip(c.xi, c.labels):
        out = (lab < 0) | (lab > 2)
        lab[out] = rng.choice(OUTSIDE, size=int(out.sum()))
        xi[:, out] = np.nan
    return c


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
def test_gpu_outside_labels(ctx, name):   # noqa: F811
    case = outside_labels(name)
    compare_blur(case, gpu_blur(ctx, case), case.oracle(), tag=name)


@pytest.mark.parametrize("name", sorted(CASES))
def test_emulated_outside_labels(name, tmp_path):
    from tests.cpu_hip import emu
    c = outside_labels(name)
    st, H, phis, taus = emu.run_blur(c.w, str(tmp_path), c.xi, c.labels, c.eps, c.G, c.H_init,
                                     c.phi_init, c.tau_init)
    assert st == 0
    compare_blur(c, (H, phis, taus), c.oracle(), tag=name)
