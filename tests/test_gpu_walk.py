"""Strips of one wave (the default schedule of large FP32 lattices with L % 4 == 0)
against the streaming plan and, for a quad, the one-kernel sweep."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_0811_2111_amd import xy

STREAM = (1, 0, 0, 1)


# 3500: the first side, cut-off tiles' place also when measured; 3720: whole strips
# (15 x 62 pairs); 4096: whole tiles when measured; 5796: past the last-level cache;
# 8192: in place of a workgroup's strips
@pytest.mark.parametrize("L", [3500, 3720, 4096, 5796, 8192])
def test_walk_matches_streaming(L):
    a = xy.Lattice(L, seed=(7 << 34) + L, beta=1.05, delta=1.1)
    b = xy.Lattice(L, seed=(7 << 34) + L, beta=1.05, delta=1.1, plan=STREAM)
    for n, every in [(1, 1), (2, 0), (5, 2)]:
        oa, ob = a.sweep(n, every), b.sweep(n, every)
        assert torch.equal(a.state, b.state), (n, every)
        if every:
            ra, rb = xy.records(oa), xy.records(ob)
            assert np.array_equal(ra["sweep"], rb["sweep"]) and np.array_equal(ra["n_accept"], rb["n_accept"])
            for f in ("cx", "cy", "ix", "iy", "mx", "my"):    # FP32 sums of a few sites, then FP64
                np.testing.assert_allclose(ra[f], rb[f], rtol=0, atol=1e-7 * L * L)


@pytest.mark.parametrize("L", [2816, 3072])       # within and past the last-level cache
def test_walk_quad_matches_one_kernel(L):
    args = ([3, 4, 1 << 40, 6], [0.7, 1.0, 1.2, 2.0], [1.0, 1.2, 0.8, 0.5])
    a, b = xy.Quad(L, *args), xy.Quad(L, *args)
    b.set_tile(32, 16)
    for n, every in [(4, 0), (5, 3)]:
        oa, ob = a.sweep(n, every), b.sweep(n, every)
        assert torch.equal(a.state, b.state), (n, every)
        if every:
            assert torch.equal(oa.view(torch.int64)[..., :2], ob.view(torch.int64)[..., :2])
