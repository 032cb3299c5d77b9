"""GPU parity of the small systems' kernels (j_stage 3) against the FP64 oracle: the fine pair tiles
(each unordered pair of one system once, in quarter sweeps shared out equally over the workgroups) and
the row groups (a workgroup finishes a few rows in one launch).

Sizes around the edges of a chunk (64 records) and a block (512), and sizes whose pieces begin inside
a sweep and cross blocks, for the row groups those of an LDS tile (1,024); every law and precision of the forces, both adjoints, the acceleration and
jerk.  A pair counted twice or missed is an error of order one in its rows.  Bars: FP64 1e-12 of the
largest value (adjoint-free paths); FP32 a median of 1e-5 and a maximum of 1e-3, on inputs rounded as
the records round them.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_0706_3060_amd import workloads as W

pytestmark = pytest.mark.gpu

FINE, FINE4, ROWS = (256, 2, 512, 1, 3), (256, 4, 1024, 1, 3), (1024, 1, 1024, 1, 3)
ROW_SIZES = [1, 2, 7, 65, 1000, 1023, 1025, 2051, 4096]
SIZES = [1, 2, 63, 65, 511, 512, 513, 1025, 2049, 5003]
ZC = (2.0e-4, -6.0e-3, 0.25, 0.4)
EPS, G = 0.01, 1.3


@pytest.fixture(scope="module")
def nb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0706_3060_amd import nbody
    return nbody


@pytest.fixture
def fine(nb):
    for api in (nb.API_FORCES, nb.API_LEAPFROG, nb.API_BACKWARD, nb.API_JERK):
        nb.set_config(api, *FINE)
    yield nb
    for api in (nb.API_FORCES, nb.API_LEAPFROG, nb.API_BACKWARD, nb.API_JERK):
        nb.clear_config(api)


def dev(a):
    return torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda")


def close(got, ref, prec):
    got = got.cpu().numpy()
    if got.ndim == 1:
        got, ref = got[:, None], ref[:, None]
    size = np.linalg.norm(ref, axis=1)
    e = np.linalg.norm(got - ref, axis=1)
    if prec == "fp64":
        assert e.max() <= 1e-12 * max(size.max(), 1e-300), e.max() / size.max()
    elif len(ref) > 1:
        e = e / np.maximum(size, 1e-3 * size.max())
        assert np.median(e) <= 1e-5 and e.max() <= 1e-3, (np.median(e), e.max())
    else:
        assert e.max() == 0.0


def sphere(n, seed):
    x, v, m = W.plummer(n, seed) if n > 1 else (np.zeros((1, 3)), np.ones((1, 3)), np.ones(1))
    return x, v, m * np.random.default_rng(seed).uniform(0.5, 1.5, n)     # unequal masses


def atoms(n, seed):
    return W.md_system(n, seed, box=(32.0 * n) ** (1.0 / 3.0) + 4.0)


def seen(prec, a):
    return a if prec == "fp64" else W.round_to_f32(a)


@pytest.mark.parametrize("cfg,n", [(FINE, n) for n in SIZES] + [(FINE4, n) for n in SIZES[2:]]
                         + [(ROWS, n) for n in ROW_SIZES])
@pytest.mark.parametrize("prec", ["fp64", "fp32_kahan", "fp32_fp64acc"])
def test_forces_of_every_law(fine, prec, cfg, n):
    nb = fine
    nb.set_config(nb.API_FORCES, *cfg)
    x, _, m = sphere(n, 900 + n)
    s = atoms(n, 800 + n)
    runs = [(nb.gravity(prec, softening=EPS, G=G), x, m,
             lambda: oracle.gravity(seen(prec, x), seen(prec, m), G=G, eps=EPS))]
    xs = seen(prec, s.pos)
    for law, ref in [(nb.ljc_linear(prec), oracle.ljc_linear), (nb.ljc_constant(prec), oracle.ljc_constant)]:
        runs.append((law, s.pos, s.params(), lambda ref=ref: ref(xs, s.q, s.sigma, s.epsilon)))
    runs.append((nb.ljc_sigmoidal(ZC, prec), s.pos, s.params(),
                 lambda: oracle.ljc_sigmoidal(xs, s.q, s.sigma, s.epsilon, ZC)))
    for law, pos, par, ref in runs:
        c = nb.get_config(nb.API_FORCES, n, law)
        four = cfg is not FINE4 or prec == "fp64" or law.kind == nb.GRAVITY      # where four i chunks are built
        assert (c["block"], c["i_per_lane"], c["j_tile"], c["j_split"], c["j_stage"]) == (cfg if four else FINE)
        f, u = nb.forces(dev(pos), dev(par), law)
        f1, u1 = nb.forces(dev(pos), dev(par), law)
        f2, _ = nb.forces(dev(pos), dev(par), law, potential=False)
        fr, ur = ref()
        close(f, fr, prec)
        close(f2, fr, prec)
        close(u, ur, prec)
        assert torch.equal(f, f1) and torch.equal(u, u1)


@pytest.mark.parametrize("n", SIZES[1:])
@pytest.mark.parametrize("prec", ["fp32_kahan", "fp32_fp64acc"])
def test_adjoints_and_jerk(fine, prec, n):
    nb = fine
    x, v, m = sphere(n, 700 + n)
    x32, v32, m32 = (W.round_to_f32(a) for a in (x, v, m))
    g = W.unit_cotangent(n, 5)
    gp, _, _ = nb.forces_backward(dev(x), dev(m), dev(g), nb.gravity(prec, softening=EPS, G=G))
    close(gp, oracle.gravity_adjoint(x32, m32, W.round_to_f32(g), G=G, eps=EPS), prec)
    a, j, p = nb.forces_jerk(dev(x), dev(v), dev(m), nb.gravity(prec, softening=EPS, G=G))
    a2, j2, _ = nb.forces_jerk(dev(x), dev(v), dev(m), nb.gravity(prec, softening=EPS, G=G), potential=False)
    for got, ref in zip((a, j, p), oracle.gravity_jerk(x32, v32, m32, G=G, eps=EPS)):
        close(got, ref, prec)
    assert torch.equal(a, a2) and torch.equal(j, j2)
    s = atoms(n, 600 + n)
    types = torch.tensor(s.types, device="cuda")
    gp, gq, gt = nb.forces_backward(dev(s.pos), dev(s.params()), dev(g), nb.ljc_linear(prec), types=types, n_types=4)
    refs = oracle.ljc_adjoint(W.round_to_f32(s.pos), s.q, s.sigma, s.epsilon, W.round_to_f32(g))
    close(gp, refs[0], prec)
    for c in range(3):
        d = np.abs(gq[:, c].cpu().numpy() - refs[1 + c]) / np.abs(refs[1 + c]).max()
        assert np.median(d) <= 1e-5 and d.max() <= 1e-3, (c, np.median(d), d.max())
    sums = np.stack([np.bincount(s.types, weights=refs[k], minlength=4) for k in (2, 3)], axis=1)
    scale = np.stack([np.bincount(s.types, weights=np.abs(refs[k]), minlength=4) for k in (2, 3)], axis=1)
    assert (np.abs(gt.cpu().numpy() - sums) <= 1e-3 * scale + 1e-300).all()


@pytest.mark.parametrize("cfg", [FINE, FINE4, ROWS])
@pytest.mark.parametrize("law,prec", [("gravity", "fp64"), ("gravity", "fp32_kahan"), ("ljc", "fp32_fp64acc"),
                                      ("ljc", "fp64")])
def test_steps_in_one_call_are_the_steps_one_by_one(fine, law, prec, cfg):
    """A step's last kernel kicks and drifts for the next step: the same arithmetic as separate calls."""
    nb = fine
    nb.set_config(nb.API_LEAPFROG, *cfg)
    n = 1333
    if law == "gravity":
        x, v, par = sphere(n, 51)
        lw, dt, im = nb.gravity(prec, softening=0.05), 1e-3, None
    else:
        s = atoms(n, 52)
        x, par, v = s.pos, s.params(), 1e-3 * np.random.default_rng(1).standard_normal((n, 3))
        lw, dt, im = nb.ljc_linear(prec), 0.5, dev(np.full(n, 3e-5))
    out = []
    for steps in ((5,), (1, 1, 1, 2)):
        X, V, P = dev(x), dev(v), dev(par)
        A = nb.forces(X, P, lw, potential=False)[0] * (im[:, None] if im is not None else 1.0)
        for k in steps:
            u = nb.leapfrog(X, V, A, P, lw, dt, k, inv_mass=im, potential=True)
        out.append((X, V, A, u))
    assert all(torch.equal(a, b) for a, b in zip(*out))


def test_rule_round_trip_and_allocation_free_call(nb):
    """The rule takes the fine tiles between the smallest systems and the coarser tiles, and for FP64; the
    reported configuration can be set; the allocation-free call gives the same sums."""
    for prec, n, want in [("fp32_kahan", 64, True), ("fp32_kahan", 4097, True), ("fp32_kahan", 9000, True), ("fp32_kahan", 32768, False), ("fp64", 9000, True),
                          ("fp64", 1 << 18, True), ("fp64", (1 << 18) + 1, False)]:
        c = nb.get_config(nb.API_FORCES, n, nb.gravity(prec))
        assert (c["j_stage"] == 3) == want, (prec, n, c)
        if want:
            nb.set_config(nb.API_FORCES, **c)
            nb.clear_config(nb.API_FORCES)
    for prec in ("fp64", "fp32_kahan"):
        for n in (1000, 9000):
            x, _, m = sphere(n, 61)
            law = nb.gravity(prec, softening=EPS)
            f, u = nb.forces(dev(x), dev(m), law)
            f1, u1 = nb.forces_noalloc(dev(x), dev(m), law)
            assert torch.equal(f, f1) and torch.equal(u, u1)


@pytest.mark.parametrize("law,prec,shape", [("gravity", "fp32_kahan", FINE4), ("ljc", "fp32_fp64acc", FINE)])
def test_the_fine_tiles_run_where_the_rule_reports_the_coarser_ones(nb, law, prec, shape):
    """33,333 particles: the rule reports j_stage 2 and the fine tiles run, bit for bit as when forced; steps
    in one call are the steps one by one there and above, where the coarser tiles run."""
    for n in (33333, 66000):
        if law == "gravity":
            x, v, par = sphere(n, 31)
            lw = nb.gravity(prec, softening=0.05)
        else:
            g = np.random.default_rng(5)
            side = int(np.ceil(n ** (1 / 3)))
            x = 3.2 * np.stack(np.unravel_index(np.arange(n), (side,) * 3), axis=1) + g.uniform(-0.3, 0.3, (n, 3))
            par = np.stack([g.uniform(-0.5, 0.5, n), np.full(n, 3.2), np.full(n, 0.1)], axis=1)
            v, lw = 1e-3 * g.standard_normal((n, 3)), nb.ljc_linear(prec)
        X, P = dev(x), dev(par)
        assert nb.get_config(nb.API_FORCES, n, lw)["j_stage"] == 2
        f, u = nb.forces(X, P, lw)
        if n <= 65536:
            nb.set_config(nb.API_FORCES, *shape)
            try:
                f2, u2 = nb.forces(X, P, lw)
            finally:
                nb.clear_config(nb.API_FORCES)
            assert torch.equal(f, f2) and torch.equal(u, u2)
        out = []
        for steps in ((3,), (1, 2)):
            Y, V, A = X.clone(), dev(v), nb.forces(X, P, lw, potential=False)[0]
            for k in steps:             # (above, the coarser tiles' shape differs with the potential)
                w = nb.leapfrog(Y, V, A, P, lw, 1e-4, k, potential=k > 1)
            out.append((Y, V, A, w))
        assert all(torch.equal(a, b) for a, b in zip(*out))
