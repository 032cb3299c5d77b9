"""Row subsets and exclusion lists use no pair tiles: a workspace of 2,048 bytes and a record a particle (the
j parts') is enough for them at every size, also where whole systems' tiles take more.
"""
import ctypes

import numpy as np
import pytest
import torch

from paper_0706_3060_amd import _native as N
from paper_0706_3060_amd import workloads as W

pytestmark = pytest.mark.gpu


def dev(a, dtype=torch.float64):
    return torch.tensor(np.asarray(a), dtype=dtype, device="cuda")


@pytest.mark.parametrize("prec,n", [("fp64", 140001), ("fp32_kahan", 40001)])
def test_subset_and_exclusions_in_a_small_workspace(prec, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0706_3060_amd import nbody as nb
    lib = N.lib()
    npad, f64 = -(-n // 64) * 64, prec == "fp64"
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    x, _, m = W.plummer(n, 3)
    X, M = dev(x), dev(m)
    rows = dev(np.arange(0, n, n // 200), torch.int64)
    law = nb.gravity(prec, softening=0.01)
    ref, refp = nb.forces_subset(X, M, rows, law)
    ws = torch.empty(npad * (2048 + (32 if f64 else 16)) + 512, dtype=torch.uint8, device="cuda")
    full = lib.nbody_workspace_bytes(0, n, 1, ctypes.byref(law.c()))
    assert full > ws.numel()
    f, p = torch.empty_like(ref), torch.empty_like(refp)
    N.check(lib.nbody_forces_subset(ptr(X), ptr(M), n, ptr(rows), rows.numel(), ctypes.byref(law.c()), ptr(f), ptr(p),
                                    ptr(ws), ws.numel(), stream))
    assert torch.equal(f, ref) and torch.equal(p, refp)
    # a whole system still needs its tiles' slots
    out = torch.empty_like(X)
    assert lib.nbody_forces(ptr(X), ptr(M), n, ctypes.byref(law.c()), ptr(out), None, ptr(ws), ws.numel(),
                            stream) == N.NBODY_EWORKSPACE
    # exclusion lists: every atom excludes the next one of its pair
    g = np.random.default_rng(5)
    side = int(np.ceil(n ** (1 / 3)))
    pos = 3.2 * np.stack(np.unravel_index(np.arange(n), (side,) * 3), axis=1) + g.uniform(-0.3, 0.3, (n, 3))
    par = np.stack([g.uniform(-0.5, 0.5, n), np.full(n, 3.2), np.full(n, 0.1)], axis=1)
    idx = np.arange(n) ^ 1
    ex = nb.Exclusions(dev(np.arange(n + 1), torch.int64), dev(np.where(idx < n, idx, n), torch.int64))
    law, Y, P = nb.ljc_linear(prec), dev(pos), dev(par)
    ref, refp = nb.forces(Y, P, law, exclusions=ex)
    ws = torch.empty(npad * (2048 + (64 if f64 else 32)) + 512, dtype=torch.uint8, device="cuda")
    f, p, e = torch.empty_like(ref), torch.empty_like(refp), ex.c(n)
    N.check(lib.nbody_forces_excl(ptr(Y), ptr(P), n, ctypes.byref(e), ctypes.byref(law.c()), ptr(f), ptr(p), ptr(ws),
                                  ws.numel(), stream))
    assert torch.equal(f, ref) and torch.equal(p, refp)


@pytest.mark.parametrize("law,prec", [("gravity", "fp64"), ("ljc", "fp64"), ("gravity", "fp32_kahan"),
                                      ("ljc", "fp32_fp64acc")])
@pytest.mark.parametrize("n,ni", [(1, 3), (63, 5), (1000, 1000), (4097, 64), (40001, 50000), (140001, 200)])
def test_the_binding_brings_no_more(law, prec, n, ni):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0706_3060_amd import nbody as nb
    g = np.random.default_rng(n)
    side = int(np.ceil(n ** (1 / 3)))
    pos = dev(3.2 * np.stack(np.unravel_index(np.arange(n), (side,) * 3), axis=1) + g.uniform(-0.3, 0.3, (n, 3)))
    lw = nb.gravity(prec, softening=0.1) if law == "gravity" else nb.ljc_linear(prec)
    par = dev(g.uniform(0.5, 1.0, n) if law == "gravity" else
              np.stack([g.uniform(-0.5, 0.5, n), np.full(n, 3.2), np.full(n, 0.1)], axis=1))
    rows = dev(g.integers(0, n, ni), torch.int64)
    nb.clear_workspace_cache()
    f, u = nb.forces_subset(pos, par, rows, lw)
    size = max(b.numel() for b in nb._ws.values())
    m = -(-max(n, ni) // 64) * 64
    assert size <= m * (2048 + (4 if law == "gravity" else 8) * (8 if prec == "fp64" else 4)) + 512
    nb.forces(pos, par, lw)                       # a larger buffer: the same sums
    f2, u2 = nb.forces_subset(pos, par, rows, lw)
    assert torch.equal(f, f2) and torch.equal(u, u2)
