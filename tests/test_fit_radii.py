"""The fits' routes by radius, against the oracle: radius 1 and 2 from the staged data, larger ones
and cells whose radius grows from global memory, bricks staged in two halves, the two fallbacks,
and the counts of all of these."""
import numpy as np
import pytest

import helpers
from cpu_hip import emu
from paper_2104_00095_amd import fields, rmx
from tests.test_fit_bricks import scattered
from tests.test_fit_halves import ball


WORKLOADS = {
    "ball": lambda: (ball((12, 12, 12)), None),
    "speck": lambda: (ball((12, 12, 12), radius=0.9, n_layers=3), None),
    "ball_spacings": lambda: (ball((12, 12, 12), spacing=(1.0, 1.3, 0.8)), None),
    "dense": lambda: (scattered((13, 9, 8), 0.25, 61), None),
    "sparse": lambda: (scattered((24, 24, 24), 0.04, 62), None),
    "plates": lambda: helpers.plates_workload(),
}
# (r_s, r_max): every first radius, without and with growth
RADII = [(1, 1), (1, 2), (1, 4), (2, 2), (2, 4), (3, 4), (4, 4)]


# A fit's error is the rounding of its sums times the condition number of its 4 x 4 system.  Smooth
# maps around a ball: up to 1e4 (FP32) and, in FP64, 1e7 over the parity bars' units; scattered
# data with the normal factor, whose weights can be small: up to 1e9.
def tolerance(name, precision):
    if precision == rmx.FP32_ACCUM:
        return 1e-3
    return 1e-9 if name.startswith("ball") else 1e-7


def compare(name, w, xn, got, radii, precision, stats=None):
    r_s, r_max = radii
    xi, lab, dec = got
    so, xo, lo, do, sto = helpers.run_oracle(w, w.solids[0], r_s=r_s, r_max=r_max,
                                             xi_normal=xn)
    assert so == 0
    assert np.array_equal(lab, lo)
    assert np.array_equal(dec, do), (name, radii, int((dec != do).sum()))
    assert helpers.rel_err(xi, xo, lo > 0) <= tolerance(name, precision)
    if stats is not None:
        band = do[lo > 0]
        code = band & 63
        want = [int((code > r_s).sum()), int((band >= 64).sum()), int((code == 32).sum()),
                int((code == 33).sum())]
        assert [stats["n_r_grown"], stats["n_no_normal"], stats["n_f1"], stats["n_f2"]] == want


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, 16])   # the launch chain, the persistent launch
@pytest.mark.parametrize("radii", RADII)
@pytest.mark.parametrize("name", sorted(WORKLOADS))
def test_gpu_radii(name, radii, flags):
    # (FP32: on the smooth maps, whose conditioning its tolerance is derived for)
    for precision in [rmx.FP64] + ([rmx.FP32_ACCUM] if name == "ball" else []):
        w, xn = WORKLOADS[name]()
        dw = fields.upload(w, decisions=True, xi_normal=None if xn is None else [xn])
        ctx = rmx.Context(0)
        st, stats = ctx.extrapolate(dw.grid, dw.solids,
                                    rmx.options(precision=precision, r_s=radii[0], r_max=radii[1],
                                                flags=flags))
        assert st == 0
        got = (dw.xi[0].cpu().numpy(), dw.labels[0].cpu().numpy(), dw.decisions[0].cpu().numpy())
        ctx.close()
        compare(name, w, xn, got, radii, precision, stats[0])


@pytest.mark.parametrize("name,radii", [("speck", (1, 4)), ("dense", (1, 4)), ("dense", (1, 1)),
                                        ("dense", (3, 4)), ("plates", (2, 4))])
def test_emulated_radii(name, radii, tmp_path):
    w, xn = WORKLOADS[name]()
    st, outs = emu.run(w, str(tmp_path), r_s=radii[0], r_max=radii[1],
                       xi_normal=None if xn is None else [xn])
    assert st == 0
    compare(name, w, xn, outs[0][:3], radii, rmx.FP64)
