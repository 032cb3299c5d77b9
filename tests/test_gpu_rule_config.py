"""The rule's configuration, reported, forced, tuned against and run through the allocation-free call, is one
kernel: from 32,768 to 65,536 particles (FP32 pair arithmetic) the rule reports the symmetric tiles'
shape for the size and runs the fine pair tiles, and setting what was reported changes nothing.
"""
import subprocess
import sys
from pathlib import Path

import numpy as np
import pytest
import torch

from paper_0706_3060_amd import workloads as W

pytestmark = pytest.mark.gpu
ROOT = str(Path(__file__).resolve().parents[1])
N = 33333


@pytest.fixture(scope="module")
def nb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0706_3060_amd import nbody
    return nbody


def dev(a):
    return torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda")


def system(nb, law, n=N):
    if law == "gravity":
        x, v, m = W.plummer(n, 31)
        return dev(x), dev(m), dev(v), nb.gravity("fp32_kahan", softening=0.05)
    g = np.random.default_rng(5)
    side = int(np.ceil(n ** (1 / 3)))
    x = 3.2 * np.stack(np.unravel_index(np.arange(n), (side,) * 3), axis=1) + g.uniform(-0.3, 0.3, (n, 3))
    par = np.stack([g.uniform(-0.5, 0.5, n), np.full(n, 3.2), np.full(n, 0.1)], axis=1)
    return dev(x), dev(par), dev(1e-3 * g.standard_normal((n, 3))), nb.ljc_linear("fp32_fp64acc")


def same(a, b):
    return all(p is None and q is None or torch.equal(p, q) for p, q in zip(a, b))


@pytest.mark.parametrize("law", ["gravity", "ljc"])
def test_setting_the_reported_configuration_changes_nothing(nb, law):
    X, P, V, lw = system(nb, law)
    g = dev(W.unit_cotangent(N, 3))

    def calls():
        A = nb.forces(X, P, lw, potential=False)[0]
        Y, Z, B = X.clone(), V.clone(), A.clone()
        u = nb.leapfrog(Y, Z, B, P, lw, 1e-4, 3, potential=True)
        gp = nb.forces_backward(X, P, g, lw)
        return [A, Y, Z, B, u, *nb.forces(X, P, lw), gp[0], gp[1]]

    ref = calls()
    apis = (nb.API_FORCES, nb.API_LEAPFROG, nb.API_BACKWARD)
    reported = [nb.get_config(api, N, lw) for api in apis]
    try:
        for api, c in zip(apis, reported):
            nb.set_config(api, **c)
            assert nb.get_config(api, N, lw) == c
        got = calls()
    finally:
        for api in apis:
            nb.clear_config(api)
    assert same(ref, got)


@pytest.mark.parametrize("n", [5000, 30011])
@pytest.mark.parametrize("api", ["API_JERK", "API_HERMITE"])
def test_setting_the_reported_jerk_configuration_leaves_shared_steps(nb, api, n):
    x, v, m = W.plummer(n, 7)
    law = nb.gravity("fp32_kahan", softening=0.02)

    def step():
        s = [dev(x), dev(v)]
        s += list(nb.forces_jerk(*s, dev(m), law, potential=False)[:2])
        nb.hermite(*s, dev(m), law, 1e-3, 2)
        return s

    ref = step()
    c = nb.get_config(getattr(nb, api), n, law)
    try:
        nb.set_config(getattr(nb, api), **c)
        got = step()
    finally:
        nb.clear_config(getattr(nb, api))
    assert same(ref, got)


@pytest.mark.parametrize("law", ["gravity", "ljc"])
def test_allocation_free_call_runs_the_same_kernel(nb, law):
    X, P, _, lw = system(nb, law)
    assert same(nb.forces(X, P, lw), nb.forces_noalloc(X, P, lw))
    assert same(nb.forces(X, P, lw, potential=False), nb.forces_noalloc(X, P, lw, potential=False))


@pytest.mark.parametrize("law", ["gravity", "ljc"])
def test_the_only_share_is_the_forces_result(nb, law):
    X, P, _, lw = system(nb, law)
    assert same(nb.forces(X, P, lw), nb.forces_share(X, P, lw, 0, 1))
    assert same(nb.forces(X, P, lw, potential=False), nb.forces_share(X, P, lw, 0, 1, potential=False))


CHILD = r"""
import sys
sys.path.insert(0, %(root)r)
sys.path.insert(0, %(root)r + "/tests")
import torch
from paper_0706_3060_amd import nbody as nb
from test_gpu_rule_config import N, same, system
X, P, V, lw = system(nb, %(law)r)
before = [nb.forces(X, P, lw), nb.forces(X[:32768], P[:32768], lw)]
cfg, ms = nb.autotune(X, P, lw)
print(cfg, ms, flush=True)
# the rule's kernel was the first candidate, so it is what a tie keeps, at every size of the bucket
assert cfg["j_stage"] == 3, cfg
after = nb.forces(X, P, lw)
nb.set_config(nb.API_FORCES, **cfg)
forced = nb.forces(X, P, lw)
nb.clear_config(nb.API_FORCES)
assert same(after, forced)
print("TUNED")
"""


@pytest.mark.parametrize("law", ["gravity", "ljc"])
def test_the_autotuner_times_the_kernel_that_the_rule_runs(law):
    # in a process of its own: a tuned entry stays until the process ends
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    r = subprocess.run([sys.executable, "-c", CHILD % dict(root=ROOT, law=law)], capture_output=True, text=True,
                       timeout=100, cwd=ROOT)
    assert r.returncode == 0 and "TUNED" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])
