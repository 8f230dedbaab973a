"""The plan that keeps a lattice in one workgroup, at the sides where a thread's share
changes (one pair up to 44, two to 62 .. 64, four to 90, eight to 128), against the
streaming plan."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_0811_2111_amd import xy

STREAM, RESIDENT = (1, 0, 0, 1), (4, 0, 0, 1)


@pytest.mark.parametrize("prec", ["fp32", "fp16"])
@pytest.mark.parametrize("L", [4, 44, 48, 64, 68, 88, 92, 100, 128])
def test_resident_plan_matches_streaming(L, prec):
    a = xy.Lattice(L, seed=(7 << 33) + L, beta=1.05, delta=1.1, precision=prec, plan=RESIDENT)
    b = xy.Lattice(L, seed=(7 << 33) + L, beta=1.05, delta=1.1, precision=prec, plan=STREAM)
    for n, every in [(1, 1), (6, 0), (13, 5)]:
        oa, ob = a.sweep(n, every), b.sweep(n, every)
        assert torch.equal(a.state, b.state), (n, every)
        if every:
            ra, rb = xy.records(oa), xy.records(ob)
            assert np.array_equal(ra["sweep"], rb["sweep"]) and np.array_equal(ra["n_accept"], rb["n_accept"])
            for f in ("cx", "cy", "ix", "iy", "mx", "my"):
                # FP32 chains of up to 16 sites with terms and sums below 32: L^2 / 32
                # chains of 16 roundings of 2^-19 at most
                np.testing.assert_allclose(ra[f], rb[f], rtol=0, atol=2.0 ** -19 * 16 * max(1.0, L * L / 32) ** 0.5 + 1e-5)
