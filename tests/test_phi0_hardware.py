"""phi0 of an ellipsoid keeps the bisection's bits whatever the reciprocals it starts from: on the
host with reciprocals off by up to 2^-22 and 2^-26, and on the GPU with the hardware's own, over
points on, near and far from the surfaces of flat, nearly round and ordinary ellipsoids."""
import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_2104_00095_amd import rmx, synth
from tests.cpu_hip import emu
from tests.helpers import oracle_shape

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "cpu_hip")


@pytest.mark.skipif(not os.path.exists(emu.CLANG), reason="no host clang++")
@pytest.mark.parametrize("bits", [22, 26])
def test_approximate_reciprocals(tmp_path, bits):
    lib = oracle.build(force=False)
    exe = str(tmp_path / "phi0_approx_check")
    subprocess.check_call([emu.CLANG, "-std=c++20", "-O2", "-Wno-unknown-attributes", "-I", HERE,
                           "-I", os.path.join(emu.ROOT, "include"), "-I", emu.CSRC,
                           "-x", "c++", os.path.join(HERE, "phi0_approx_check.cpp"), "-x", "none",
                           lib, "-Wl,-rpath," + os.path.dirname(lib), "-o", exe])
    out = subprocess.run([exe, "200000", str(bits)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout + out.stderr


SEMI = {"ordinary": (0.3, 0.2, 0.25), "flat": (0.3, 0.28, 0.004), "needle": (0.4, 0.01, 0.012),
        "nearly_round": (0.25, 0.25 * (1 + 1e-15), 0.25 * (1 + 1e-9)), "round": (0.2, 0.2, 0.2),
        "large": (3e5, 1e5, 2e5), "small": (3e-7, 1e-7, 2e-7)}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(SEMI))
def test_gpu_bits(name):
    """phi of a box whose map holds the points, every cell covered: bit for bit the oracle's."""
    import torch
    rng = np.random.default_rng(5)
    n = 40
    semi = np.array(SEMI[name])
    shape = synth.ellipsoid_shape(tuple(0.3 * semi), tuple(semi), synth.random_rotation(rng))
    rot = np.asarray(shape.rot).reshape(3, 3)
    d = rng.standard_normal((3, n ** 3))
    d /= np.linalg.norm(d, axis=0)
    # a third each: on the surface to rounding, close to it on all scales, anywhere about
    off = 10.0 ** (-10.0 * rng.random(n ** 3)) * rng.choice([-1.0, 1.0], n ** 3)
    kind = np.arange(n ** 3) % 3
    scale = np.where(kind == 0, 1.0, np.where(kind == 1, 1.0 + off, 3.0 * rng.random(n ** 3)))
    xi = (0.3 * semi)[:, None] + rot @ (d * semi[:, None] * scale)
    xi = np.ascontiguousarray(xi.reshape(3, n, n, n))
    lab = np.zeros((n, n, n), dtype=np.int8)
    eps = 0.1 * float(semi.min())
    T = lambda a: torch.from_numpy(a).to("cuda")
    phi = torch.full((n, n, n), -6.0, dtype=torch.float64, device="cuda")
    ctx = rmx.Context(0)
    g = rmx.grid((n, n, n), 1.0 / n, (0.0, 0.0, 0.0))
    s = rmx.solid((0, 0, 0), (n, n, n), rmx.shape(shape.kind, shape.centre, shape.semi, shape.rot),
                  1, T(xi), T(lab))
    ctx.blur(g, [s], eps, None, [phi])
    torch.cuda.synchronize()
    ctx.close()
    _, want = oracle.blur((n, n, n), [((0, 0, 0), (n, n, n), oracle_shape(shape), 1, xi, lab)], eps,
                          np.ones((n, n, n)), [np.zeros((n, n, n))])
    got = phi.cpu().numpy()
    assert np.array_equal(got.view(np.uint64), want[0].view(np.uint64)), \
        int((got.view(np.uint64) != want[0].view(np.uint64)).sum())
