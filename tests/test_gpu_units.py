"""FP32 gravity in SI units (a star cluster: metres, kilograms, seconds), where the inverse cube of a
distance, 1e-50, is far below FP32 but m / s and 1 / s^2 are not.  Row groups, fine pair tiles with two
and four i chunks, leapfrog and shared Hermite steps against the FP64 law: FP32 pair terms, a median of 1e-5 and a
maximum of 1e-3 of a row's size.
"""
import numpy as np
import pytest
import torch

from paper_0706_3060_amd import workloads as W

pytestmark = pytest.mark.gpu

PARSEC, SUN, G_SI = 3.0857e16, 1.989e30, 6.674e-11


@pytest.fixture(scope="module")
def nb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0706_3060_amd import nbody
    return nbody


def dev(a):
    return torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda")


def cluster(n):
    x, v, m = W.plummer(n, 12)
    # total mass n suns, the length unit one parsec: the velocity unit follows from G
    speed = np.sqrt(G_SI * n * SUN / PARSEC)
    # as the records round them
    x, v, m = (W.round_to_f32(a) for a in (x * PARSEC, v * speed, m * n * SUN))
    return dev(x), dev(v), dev(m), PARSEC / speed


def close(got, ref):
    if got.dim() == 1:
        got, ref = got[:, None], ref[:, None]
    e = ((got - ref).norm(dim=1) / ref.norm(dim=1)).cpu().numpy()
    assert np.isfinite(e).all() and np.median(e) <= 1e-5 and e.max() <= 1e-3, (np.median(e), e.max())


@pytest.mark.parametrize("n", [1000, 5003, 30011])
@pytest.mark.parametrize("prec", ["fp32_kahan", "fp32_fp64acc"])
def test_forces_and_steps_in_si_units(nb, prec, n):
    x, v, m, time = cluster(n)
    laws = [nb.gravity(p, softening=0.01 * PARSEC, G=G_SI) for p in (prec, "fp64")]
    (f, u), (fr, ur) = (nb.forces(x, m, law) for law in laws)
    close(f, fr)
    close(u, ur)
    close(nb.forces(x, m, laws[0], potential=False)[0], fr)
    out = []
    for law in laws:
        X, V, A = x.clone(), v.clone(), fr.clone()
        nb.leapfrog(X, V, A, m, law, 1e-3 * time, 2)
        A0, J0, _ = nb.forces_jerk(x, v, m, laws[1], potential=False)
        Y, Z, B, J = x.clone(), v.clone(), A0.clone(), J0.clone()
        nb.hermite(Y, Z, B, J, m, law, 1e-3 * time, 1)
        out.append((X, V, A, Y, Z, B, J))
    for got, ref in zip(*out):
        close(got, ref)
