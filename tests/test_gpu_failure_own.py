"""Injected launch failures at every launch point of the library's own schedules: the
counter, the angles and the records of the sweeps done before, then the rest of the
trajectory."""
from __future__ import annotations

import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_0811_2111_amd import xy


def counts(rec):
    return rec.view(torch.int64)[..., :2]


def lattice(L):
    return xy.Lattice(L, seed=77, beta=1.1, delta=1.0)


def quad(L):
    return xy.Quad(L, [3, 4, 1 << 40, 6], [0.7, 1.0, 1.2, 2.0])


# kept: whether the records of all sweeps done are written (those of passes are
# reduced together, a failed reduction is made up for; a single sweep's record is lost
# with its reduction)
@pytest.mark.parametrize("make,L,n,every,kept", [
    ("lattice", 256, 20, 2, True), ("lattice", 1002, 13, 3, True), ("lattice", 1202, 6, 2, False),
    ("lattice", 3500, 5, 2, False), ("quad", 64, 9, 1, True), ("quad", 96, 9, 3, True), ("quad", 544, 9, 3, True),
    ("quad", 864, 9, 3, False), ("quad", 864, 4, 1, False)])
def test_failure_at_every_launch_point(make, L, n, every, kept):
    make = globals()[make]
    ref, failed = make(L), 0
    want = ref.sweep(n, every)
    for after in range(1000):
        h = make(L)
        out = torch.full_like(want, -1.0)
        xy.xy_test_inject_failure(after)
        try:
            h.sweep(n, every, out=out)
            break                                      # beyond the last launch point
        except xy.XYError as e:
            assert e.code == xy.XY_EHIP
        finally:
            xy.xy_test_inject_failure(-1)
        failed += 1
        s = h.sweep_count
        done = s // every if kept else max(0, s // every - 1)
        assert torch.equal(counts(out[:done]), counts(want[:done])), after
        assert torch.allclose(out[:done, ..., 2:], want[:done, ..., 2:], rtol=0, atol=2.0 ** -52 * 8 * L * L), after
        h.sweep(n - s)
        assert torch.equal(h.state, ref.state) and h.sweep_count == n, after
    assert failed >= 3


@pytest.mark.parametrize("make,L", [("lattice", 64), ("quad", 64)])
def test_hmc_failure_at_every_launch_point(make, L):
    """Trajectories that are rejected: the angles are those before them."""
    make = globals()[make]
    for eps in (0.1, 2.5):
        for after in range(100):
            h, ref = make(L), make(L)
            xy.xy_test_inject_failure(after)
            try:
                h.hmc(3, 7, eps)
                break
            except xy.XYError as e:
                assert e.code == xy.XY_EHIP
            finally:
                xy.xy_test_inject_failure(-1)
            if h.sweep_count:
                ref.hmc(h.sweep_count, 7, eps)
            assert torch.equal(h.state, ref.state), (eps, after)
        assert after >= 4                              # three trajectories and what follows them
