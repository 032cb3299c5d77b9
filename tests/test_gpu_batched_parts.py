"""GPU parity of the batched symmetric tiles in 1, 2 and 4 parts (a wave for each part of a tile's j
chunks), forward and backward, against the FP64 oracle: sizes around the chunk (64) and block (256) edges, where parts of a
system's last block hold only padding, and systems long enough that the workspace holds 2 parts or 1.
A slot missed or added twice is an error of order one in its rows; the bars are those of the tiles
themselves (FP32 sums: a median of 1e-5 and a maximum of 1e-3 of a row's size).
"""
import numpy as np
import pytest
import torch

import test_gpu_batched_symmetric_adjoint as adjoint
from paper_0706_3060_amd import workloads as W
from test_gpu_batched_symmetric import BSYM, check_system, ensemble, gpu_law, host, nb, run  # noqa: F401

pytestmark = pytest.mark.gpu

FOUR = [1, 2, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 320, 321, 449, 0, 705, 1025]
TWO = [3841, 3905, 4033]         # 16 blocks: the region of 32 slots a row holds 2 parts
ONE = [8192]


@pytest.mark.parametrize("potential", [True, False])
@pytest.mark.parametrize("law", ["gravity", "ljc_linear"])
@pytest.mark.parametrize("sizes", [FOUR, TWO, ONE], ids=["four", "two", "one"])
def test_parts_of_a_tile(nb, sizes, law, potential):  # noqa: F811
    off, x, par = ensemble(law, sizes, 41)
    lw = gpu_law(nb, law, "fp32_kahan")
    out = [run(nb, off, x, par, lw, potential, BSYM) for _ in range(2)]
    (f, p), (f2, p2) = out
    assert torch.equal(f, f2) and (p is None or torch.equal(p, p2))
    f, p = host(f), None if p is None else host(p)
    for s in range(len(sizes)):
        a, b = int(off[s]), int(off[s + 1])
        check_system(law, x[a:b], par[a:b], f[a:b], None if p is None else p[a:b], potential)
    assert np.isfinite(f).all()


@pytest.mark.parametrize("law", ["gravity", "ljc_linear"])
@pytest.mark.parametrize("sizes", [FOUR, TWO, ONE], ids=["four", "two", "one"])
def test_parts_of_an_adjoint_tile(nb, sizes, law):  # noqa: F811
    off, x, par, types = adjoint.ensemble(law, sizes, 43)
    g = W.unit_cotangent(x.shape[0], 44)
    lw = adjoint.gpu_law(nb, law, "fp32_kahan")
    one, two = (adjoint.backward(nb, off, x, par, g, lw, adjoint.BSYM) for _ in range(2))
    gp, gq = host(one[0]), None if law == "gravity" else host(one[1])
    assert torch.equal(one[0], two[0]) and (gq is None or torch.equal(one[1], two[1]))
    for s in range(len(sizes)):
        a, b = int(off[s]), int(off[s + 1])
        adjoint.check_system(law, x[a:b], par[a:b], g[a:b], gp[a:b], None if gq is None else gq[a:b])
