"""A weight of the blur zone can round to just above 1 (1 - H_eps a last bit above it, close to
phi = -eps), also of the one solid that covers a face: the blend then divides by it, as it does by
any sum above 1.  On the CPU, where the sine is the oracle's, the stress equals the oracle's bit
for bit."""
import numpy as np

import oracle
from paper_2104_00095_amd import synth
from tests.cpu_hip import emu
from tests.helpers import BlurCase, oracle_shape


def patch(n=12, seed=3):
    """A box that lies within 2e-6 eps of the surface phi = -eps of a ball, every cell covered."""
    rng = np.random.default_rng(seed)
    h = 1.0 / n
    w = synth.Workload("patch", (n, n, n), h, (0.0, 0.0, 0.0))
    x, y, z = synth.cell_centres((0, 0, 0), (n, n, n), h, (0.0, 0.0, 0.0))
    X = np.stack(np.broadcast_arrays(x, y, z)) - 0.5
    e = rng.standard_normal(3)
    at = (0.4 - 0.1 * (1.0 - 1e-6)) * e / np.linalg.norm(e)
    A = 5e-8 * (np.eye(3) + 0.3 * rng.standard_normal((3, 3)))
    xi = np.ascontiguousarray(at[:, None, None, None] + np.einsum("ab,bkji->akji", A, X))
    w.solids.append(synth.Solid((0, 0, 0), (n, n, n), synth.sphere_shape((0.0, 0.0, 0.0), 0.4), 2,
                                xi))
    c = BlurCase.__new__(BlurCase)
    c.w, c.eps, c.xi, c.labels, c.G = w, 0.1, [xi], [np.zeros((n, n, n), np.int8)], [1.0]
    c.H_init = np.full((n, n, n), 5.0)
    c.phi_init = [np.full((n, n, n), -6.0)]
    c.tau_init = [np.full((6, n + (a == 2), n + (a == 1), n + (a == 0)), 7.0) for a in range(3)]
    return c


def test_emulated_weight_above_one(tmp_path):
    c = patch()
    s = c.w.solids[0]
    mid = 0.5 * (c.xi[0][:, :, :, 1:] + c.xi[0][:, :, :, :-1])
    shape = oracle_shape(s.shape)
    above = 0
    for k, j, i in np.ndindex(mid.shape[1:]):
        above += 1.0 - oracle.heaviside_eps(oracle.phi0(shape, mid[:, k, j, i]), c.eps) > 1.0
    assert above > 0
    st, H, phis, taus = emu.run_blur(c.w, str(tmp_path), c.xi, c.labels, c.eps, c.G, c.H_init,
                                     c.phi_init, c.tau_init)
    assert st == 0
    for got, want in zip(taus, c.oracle()[2]):
        assert np.array_equal(got, want), int((got != want).sum())
