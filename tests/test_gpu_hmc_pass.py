"""Leap-frog passes in registers on any even lattice against one step per launch,
and batches of such lattices against single ones."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_0811_2111_amd import xy

# 4, 6: a region holds many copies of the lattice; 112, 114: one core of 56 entries
# and the first that needs a second; 130, 1002: an odd number of entries a row;
# 640 .. 832: where regions change from four rows a thread to eight
SIZES = [4, 6, 34, 112, 114, 130, 640, 770, 832, 1000, 1002]


@pytest.mark.parametrize("L", SIZES)
def test_passes_match_single_steps(L):
    ref = None
    for steps in (1, 2, 7, 8):
        lat = xy.Lattice(L, seed=(3 << 33) + L, beta=1.05)
        lat.set_hmc_steps_per_pass(steps)
        rec = xy.hmc_records(lat.hmc(2, 9, 0.15))          # a short last pass
        rej = xy.hmc_records(lat.hmc(1, 8, 2.5))
        got = (lat.state.clone(), rec.tobytes(), rej.tobytes())
        if ref is None:
            ref = got
        else:
            assert torch.equal(got[0], ref[0]) and got[1:] == ref[1:], steps


@pytest.mark.parametrize("Ls", [[100, 36, 64, 4], [1000, 512, 1024, 20]])
def test_batches_of_any_side_match_single_lattices(Ls):
    """Few regions (four rows a thread) and many (eight)."""
    n = len(Ls)
    seeds, betas = [11 + i for i in range(n)], [0.9 + 0.1 * i for i in range(n)]
    for steps in (7, 1):
        b = xy.Batch(Ls, seeds, betas, [1.0] * n)
        b.set_hmc_steps_per_pass(steps)
        rec = xy.hmc_records(b.hmc(2, 10, 0.1))
        for i, L in enumerate(Ls):
            lat = xy.Lattice(L, seed=seeds[i], beta=betas[i])
            srec = xy.hmc_records(lat.hmc(2, 10, 0.1))
            assert srec.tobytes() == rec[i].tobytes() and torch.equal(b.lattice_state(i), lat.state), (steps, L)


@pytest.mark.parametrize("L", [32, 34, 64, 300])
def test_several_trajectories_a_call_match_single_calls(L):
    """Rejected trajectories are undone by the next one of the call, the last by the call."""
    a, b = (xy.Lattice(L, seed=(5 << 33) + L, beta=1.05) for _ in range(2))
    seen = set()
    for eps in (0.05, 0.2, 0.35, 2.5):
        many = xy.hmc_records(a.hmc(6, 7, eps))
        one = [xy.hmc_records(b.hmc(1, 7, eps)) for _ in range(6)]
        assert many.tobytes() == b"".join(r.tobytes() for r in one) and torch.equal(a.state, b.state), eps
        seen |= set(int(v) for v in many["accepted"])
    assert seen == {0, 1}
    if L % 32 == 0:
        args = ([1, 2, 3, 4], [0.7, 0.9, 1.1, 1.3])
        a, b = xy.Quad(L, *args), xy.Quad(L, *args)
        for eps in (0.05, 0.2, 0.35, 2.5):
            many = xy.hmc_records(a.hmc(6, 7, eps))
            one = [xy.hmc_records(b.hmc(1, 7, eps)) for _ in range(6)]
            assert many.tobytes() == b"".join(r.tobytes() for r in one) and torch.equal(a.state, b.state), eps


def test_injected_failure_between_trajectories():
    ref = xy.Lattice(64, seed=9, beta=1.1)
    ref.hmc(2, 7, 2.5)                                     # rejected
    lat = xy.Lattice(64, seed=9, beta=1.1)
    xy.xy_test_inject_failure(2)
    try:
        with pytest.raises(xy.XYError):
            lat.hmc(4, 7, 2.5)
    finally:
        xy.xy_test_inject_failure(-1)
    assert lat.sweep_count == 2 and torch.equal(lat.state, ref.state)
