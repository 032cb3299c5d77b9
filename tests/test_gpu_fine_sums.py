"""Sums of the fine pair tiles (j_stage 3) below 32,768 particles: FP32 pair terms are added as FP32 chains
of at most 256, as the one-sided kernels add them, and everything after a chain is FP64.

Three sources at one place with masses 2^24, 1 and -2^24 act on massless particles at another: every pair
term is exact in FP32 (the softening is 1, the offset 2^-13 or 0, so s rounds to 1), the three lie in
chains of their own, and the sum is the small source's term.  A partial sum held in FP32 anywhere past
the chains loses it whole (2^24 + 1 rounds to 2^24), so the error is 1; with FP64 it is the pair terms'
own rounding, below 1e-6.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

N, D = 5000, 2.0 ** -13
# rows of the sources: j sums of one block meet across its waves (0 and 256 lie in waves of their own in
# a block of 512 or 1,024 rows); i sums of one workgroup meet across neighbouring chunks of 64
SOURCES = {"j": (0, 256, 1024), "i": (2303, 2304, 4096)}


@pytest.fixture(scope="module")
def nb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0706_3060_amd import nbody
    return nbody


def dev(a):
    return torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda")


def setup(side, shift):
    rows = list(SOURCES[side])
    pos, mass = np.zeros((N, 3)), np.zeros(N)
    mass[rows] = 2.0 ** 24, 1.0, -(2.0 ** 24)
    pos[rows, 0] = shift
    probes = np.arange(2048, N) if side == "j" else np.arange(0, 1024)
    return pos, mass, rows, probes


@pytest.mark.parametrize("side", ["j", "i"])
@pytest.mark.parametrize("cfg", [None, (256, 2, 512, 1, 3), (256, 4, 1024, 1, 3)])
@pytest.mark.parametrize("prec", ["fp32_kahan", "fp32_fp64acc"])
def test_forces(nb, prec, cfg, side):
    pos, mass, rows, probes = setup(side, D)
    law = nb.gravity(prec, softening=1.0)
    assert nb.get_config(nb.API_FORCES, N, law)["j_stage"] == 3
    if cfg:
        nb.set_config(nb.API_FORCES, *cfg)
    try:
        f, u = nb.forces(dev(pos), dev(mass), law)
    finally:
        nb.clear_config(nb.API_FORCES)
    assert np.abs(f.cpu().numpy()[probes] / D - np.array([1.0, 0.0, 0.0])).max() <= 1e-6
    assert np.abs(u.cpu().numpy()[probes] + 1.0).max() <= 1e-6


@pytest.mark.parametrize("side", ["j", "i"])
@pytest.mark.parametrize("prec", ["fp32_kahan", "fp32_fp64acc"])
def test_position_adjoint(nb, prec, side):
    # without an offset the pair's Hessian is minus the identity: the gradient of a massless
    # particle with cotangent e_y is minus the sum of the masses, in y
    pos, mass, rows, probes = setup(side, 0.0)
    law = nb.gravity(prec, softening=1.0)
    assert nb.get_config(nb.API_BACKWARD, N, law)["j_stage"] == 3
    g = np.zeros((N, 3))
    g[probes, 1] = 1.0
    gp, _, _ = nb.forces_backward(dev(pos), dev(mass), dev(g), law)
    assert np.abs(gp.cpu().numpy()[probes] - np.array([0.0, -1.0, 0.0])).max() <= 1e-6


@pytest.mark.parametrize("side", ["j", "i"])
@pytest.mark.parametrize("prec", ["fp32_kahan", "fp32_fp64acc"])
def test_shared_hermite_step(nb, prec, side):
    # a short step leaves the new acceleration and jerk in acc and jerk: with the sources moving at e_y
    # the jerk of a massless particle at rest is the sum of the masses, in y
    pos, mass, rows, probes = setup(side, D)
    vel = np.zeros((N, 3))
    vel[rows, 1] = 1.0
    X, V, A, J = dev(pos), dev(vel), dev(np.zeros((N, 3))), dev(np.zeros((N, 3)))
    nb.hermite(X, V, A, J, dev(mass), nb.gravity(prec, softening=1.0), 2.0 ** -30, 1)
    assert np.abs(A.cpu().numpy()[probes, 0] / D - 1.0).max() <= 1e-6
    # (d.w) d and the drift of the sources, 2^-30 and 2^-43, are below the bar
    assert np.abs(J.cpu().numpy()[probes] - np.array([0.0, 1.0, 0.0])).max() <= 1e-6
