"""Single-sweep tiles on lattices that they do not divide (the default schedule
beyond the small lattices) against the streaming plan."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_0811_2111_amd import xy

STREAM = (1, 0, 0, 1)
# 258: a measured single sweep of a lattice with one entry left for the second tile;
# 834, 1002: L % 4 == 2 (a last pair of one entry), 836, 900: L % 4 == 0, the last tile
# of 68 and 4 columns, 4 rows; 1410, 1412: 128 and 256 columns a tile; 2050: two
# columns left; 2304: whole tiles of another shape than the reported plan's
SIZES = [258, 834, 836, 900, 1002, 1410, 1412, 2050, 2304]


@pytest.mark.parametrize("prec", ["fp32", "fp16"])
@pytest.mark.parametrize("L", SIZES)
def test_ragged_tiles_match_streaming(L, prec):
    a = xy.Lattice(L, seed=(9 << 33) + L, beta=1.05, delta=1.1, precision=prec)
    b = xy.Lattice(L, seed=(9 << 33) + L, beta=1.05, delta=1.1, precision=prec, plan=STREAM)
    for n, every in [(1, 1), (2, 0), (5, 2), (3, 3)]:
        oa, ob = a.sweep(n, every), b.sweep(n, every)
        assert torch.equal(a.state, b.state), (n, every)
        if every:
            ra, rb = xy.records(oa), xy.records(ob)
            assert np.array_equal(ra["sweep"], rb["sweep"]) and np.array_equal(ra["n_accept"], rb["n_accept"])
            for f in ("cx", "cy", "ix", "iy", "mx", "my"):    # FP32 sums of a few sites, then FP64
                np.testing.assert_allclose(ra[f], rb[f], rtol=0, atol=1e-7 * L * L)


def test_ragged_tiles_nontemporal_stores():
    """A lattice whose two buffers exceed the last-level cache: two sweeps."""
    L = 5830
    a = xy.Lattice(L, seed=5, beta=1.0, delta=1.2)
    b = xy.Lattice(L, seed=5, beta=1.0, delta=1.2, plan=STREAM)
    ra, rb = xy.records(a.sweep(2, 2)), xy.records(b.sweep(2, 2))
    assert torch.equal(a.state, b.state) and np.array_equal(ra["n_accept"], rb["n_accept"])


def test_injected_failure_on_ragged_tiles():
    L, n = 1202, 6
    ref = xy.Lattice(L, seed=77, beta=1.1, delta=1.0)
    ref.sweep(n, 2)
    for after in (0, 1, 3, 7):
        lat = xy.Lattice(L, seed=77, beta=1.1, delta=1.0)
        xy.xy_test_inject_failure(after)
        try:
            with pytest.raises(xy.XYError):
                lat.sweep(n, 2)
        finally:
            xy.xy_test_inject_failure(-1)
        lat.sweep(n - lat.sweep_count)
        assert torch.equal(lat.state, ref.state) and lat.sweep_count == n, after
