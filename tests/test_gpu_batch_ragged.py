"""Batches whose sides share no large tile shape (tiles that need not divide the
lattices) against the batch's own shape and against single lattices."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_0811_2111_amd import xy

STREAM = (1, 0, 0, 1)
# 36, 60: smaller than a tile; 64, 256: whole tiles of either width; 516, 1028: four
# columns left of a wide tile; 24: held on chip; 32, 96, 128: a 32 x 16 batch
BATCHES = [[100, 200, 400], [36, 60, 64, 100], [24, 256, 512, 1000], [4, 260, 516, 1028], [32, 96, 128, 192]]


@pytest.mark.parametrize("prec", ["fp32", "fp16"])
@pytest.mark.parametrize("Ls", BATCHES)
def test_ragged_batch_matches_its_own_shape_and_single_lattices(Ls, prec):
    n = len(Ls)
    seeds, betas = [5 + i for i in range(n)], [0.9 + 0.1 * i for i in range(n)]
    a = xy.Batch(Ls, seeds, betas, [1.1] * n, precision=prec)
    b = xy.Batch(Ls, seeds, betas, [1.1] * n, precision=prec)
    b.set_tile(*b.tile)                      # asked for: the shape that divides every side
    total = 0
    for sweeps, every in [(1, 1), (4, 0), (7, 3)]:       # odd and even pass counts
        oa, ob = a.sweep(sweeps, every), b.sweep(sweeps, every)
        assert torch.equal(a.state, b.state), (sweeps, every)
        if every:
            ra, rb = xy.records(oa), xy.records(ob)
            assert np.array_equal(ra["sweep"], rb["sweep"]) and np.array_equal(ra["n_accept"], rb["n_accept"])
            for f in ("cx", "cy", "ix", "iy", "mx", "my"):    # the same FP32 terms, FP64 sums in another order
                np.testing.assert_allclose(ra[f], rb[f], rtol=0, atol=1e-12 * max(Ls) ** 2)
        total += sweeps
    for i, L in enumerate(Ls):
        lat = xy.Lattice(L, seed=seeds[i], beta=betas[i], delta=1.1, precision=prec, plan=STREAM)
        lat.sweep(total)
        assert torch.equal(lat.state, a.lattice_state(i)), L
