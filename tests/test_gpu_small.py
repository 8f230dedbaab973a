"""The default schedules of small lattices (the whole lattice in one workgroup, then
several sweeps per launch on overlapping regions) against the streaming plan, at
the sizes where they change over and where regions, rows and pairs come out uneven."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_0811_2111_amd import xy

STREAM = (1, 0, 0, 1)
# 4, 6: one pair a row, two pairs with one entry missing; 32, 34: the last size of a
# workgroup of 512 and the first beyond it; 54, 56, 58: the change-over and its
# L % 4 == 2 neighbours; 256, 258: 16 x 16 sites a region and the first uneven
# split; 512: two pairs a thread; 800, 834, 1002: four; 576, 640, 832, 1088: cores of
# whole blocks of rows for the records; 1100, 1102: the last size of several sweeps a launch
SIZES = [4, 6, 32, 34, 54, 56, 58, 128, 256, 258, 386, 512, 576, 640, 800, 832, 834, 1002, 1088, 1100, 1102]


@pytest.mark.parametrize("prec", ["fp32", "fp16"])
@pytest.mark.parametrize("L", SIZES)
def test_default_schedule_matches_streaming(L, prec):
    a = xy.Lattice(L, seed=(7 << 33) + L, beta=1.05, delta=1.1, precision=prec)
    b = xy.Lattice(L, seed=(7 << 33) + L, beta=1.05, delta=1.1, precision=prec, plan=STREAM)
    for n, every in [(2, 0), (1, 1), (13, 5), (17, 1)]:       # odd and even pass counts, records inside a pass
        oa, ob = a.sweep(n, every), b.sweep(n, every)
        assert torch.equal(a.state, b.state), (n, every)
        if every:
            ra, rb = xy.records(oa), xy.records(ob)
            assert np.array_equal(ra["sweep"], rb["sweep"]) and np.array_equal(ra["n_accept"], rb["n_accept"])
            for f in ("cx", "cy", "ix", "iy", "mx", "my"):    # FP32 sums of a few sites, then FP64
                np.testing.assert_allclose(ra[f], rb[f], rtol=0, atol=1e-7 * L * L)
    assert a.sweep_count == b.sweep_count


@pytest.mark.parametrize("L", [32, 256])
def test_default_schedule_after_an_injected_failure(L):
    ref = xy.Lattice(L, seed=77, beta=1.1, delta=1.0)
    ref_obs = xy.records(ref.sweep(40, 2))
    for after in range(0, 1 if L < 56 else 11, 3):
        lat = xy.Lattice(L, seed=77, beta=1.1, delta=1.0)
        xy.xy_test_inject_failure(after)
        try:
            with pytest.raises(xy.XYError):
                lat.sweep(40, 2)
        finally:
            xy.xy_test_inject_failure(-1)
        s = lat.sweep_count
        s += s % 2 and lat.sweep(1) is None                    # continue at a record's sweep
        rest = xy.records(lat.sweep(40 - s, 2)) if s < 40 else []
        assert torch.equal(lat.state, ref.state) and lat.sweep_count == 40, after
        for r, q in zip(rest, ref_obs[s // 2:]):
            assert int(r["sweep"]) == int(q["sweep"]) and int(r["n_accept"]) == int(q["n_accept"])
