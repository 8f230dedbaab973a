"""Calls that are split into several launches, against the same sweeps in short calls."""
from __future__ import annotations

import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_0811_2111_amd import xy

STREAM = (1, 0, 0, 1)


@pytest.mark.parametrize("L,n,every", [(54, 400_000, 1000), (54, 400_000, 390_000), (54, 740_000, 369_000)])
def test_records_across_the_launches_of_a_long_call(L, n, every):
    """368 225 sweeps a launch at most: cut at records, or inside a longer interval."""
    a, b = (xy.Lattice(L, seed=3, beta=1.0, delta=1.1) for _ in range(2))
    out = a.sweep(n, every)
    one = torch.cat([b.sweep(every, every) for _ in range(n // every)])
    b.sweep(n - n // every * every)
    assert torch.equal(out.view(torch.int64), one.view(torch.int64)) and torch.equal(a.state, b.state)


def test_record_interval_beyond_the_call():
    """No record, the sweeps of an unmeasured call, nothing written through the pointer."""
    out = torch.full((1, 8), 7.0, dtype=torch.float64, device="cuda")
    for h, ref in ((xy.Lattice(32, seed=3), xy.Lattice(32, seed=3, plan=STREAM)),
                   (xy.Quad(32, [1, 2, 3, 4], [1.0] * 4), xy.Quad(32, [1, 2, 3, 4], [1.0] * 4))):
        fn = xy.lib().xy_sweep if isinstance(h, xy.Lattice) else xy.lib().xy_quad_sweep
        assert fn(h.h, 3, 2 ** 31 - 1, out.data_ptr()) == xy.XY_OK
        ref.sweep(3)
        assert torch.equal(h.state, ref.state) and h.sweep_count == 3 and bool((out == 7.0).all())
