"""Workspace sizes (host only): what the fine pair tiles (j_stage 3) add to FP64 forces and leapfrog calls.

A one-sided call needs the records and up to 64 j parts of 32 bytes a particle.  The fine tiles' slots are
reused from that space up to 131,072 particles but for the workgroups' own rows (at most 35 MB), and
reach twice that space at 262,144, the largest system they take.
"""
import ctypes

import pytest

from paper_0706_3060_amd import _native as N


@pytest.mark.parametrize("kind,record", [(0, 32), (1, 64), (2, 64), (3, 64)])
@pytest.mark.parametrize("api", [0, 3])
def test_fp64_workspace_against_the_j_parts(api, kind, record):
    law = N.NBodyLaw(kind, 0, 1.0, 0.01, 332.0637, 4.0)
    for n in (1, 100, 2049, 4097, 8192, 12001, 20480, 32768, 32769, 50001, 100000, 1 << 17, (1 << 17) + 1, 200001,
              1 << 18, (1 << 18) + 1, 1 << 19):
        npad = -(-n // 64) * 64
        parts = max(1, min(64, npad // 64, (1 << 25) // npad))
        one_sided = npad * (record + parts * 32 + (24 if api == 3 else 0))
        w = N.lib().nbody_workspace_bytes(api, n, 1, ctypes.byref(law))
        most = 2.0 * one_sided if 1 << 17 < n <= 1 << 18 else one_sided
        assert w <= 1.05 * most + (40 << 20), (n, w / one_sided)
        assert w >= one_sided
        if n > 1 << 18:
            assert w <= one_sided + 1024, n
