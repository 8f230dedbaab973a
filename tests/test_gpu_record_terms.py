"""Records of the library's own schedules against those of the plan that xy_get_plan
reports, asked for by name: the same FP32 terms, in FP64 sums of another order."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_0811_2111_amd import xy

STREAM = (1, 0, 0, 1)


def assert_same_terms(L, plan, prec="fp32"):
    a = xy.Lattice(L, seed=(5 << 33) + L, beta=1.05, delta=1.1, precision=prec)
    b = xy.Lattice(L, seed=(5 << 33) + L, beta=1.05, delta=1.1, precision=prec, plan=plan or a.plan)
    for n, every in [(1, 1), (7, 2), (12, 1)] if L < 3000 else [(1, 1), (3, 2)]:
        ra, rb = xy.records(a.sweep(n, every)), xy.records(b.sweep(n, every))
        assert np.array_equal(ra["sweep"], rb["sweep"]) and np.array_equal(ra["n_accept"], rb["n_accept"])
        for f in ("cx", "cy", "ix", "iy", "mx", "my"):
            # L^2 / 4 pairs of terms below 8 each: a misplaced or reordered FP32 term
            # shows, the order of the FP64 sums does not
            np.testing.assert_allclose(ra[f], rb[f], rtol=0, atol=2.0 ** -52 * 8 * L * L, err_msg="%s %d" % (f, n))


# one workgroup (4, 54, 62 with one sweep), several sweeps per launch in all their
# forms of columns (128, 576, 704, 768, 832) and pair by pair (58, 386, 1002), tiles
# that do not divide the lattice (836, 1202, 2050), tiles between strips of one wave (4224)
@pytest.mark.parametrize("prec", ["fp32", "fp16"])
@pytest.mark.parametrize("L", [4, 54, 62, 58, 128, 386, 576, 704, 768, 832, 836, 1002, 1202, 2050, 4224])
def test_records_gather_the_reported_plans_terms(L, prec):
    assert_same_terms(L, None, prec)


# strips of one wave, also where the reported plan is a tile (3520: 64 x 32, 7296:
# 128 x 32), whose columns they do not gather
@pytest.mark.parametrize("L", [3500, 3520, 5796, 7296])
def test_strip_records_gather_pairs(L):
    assert_same_terms(L, STREAM)
