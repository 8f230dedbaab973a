"""Calls captured into a graph and replayed, with the state put back and other work of
the program in between, against the same calls run eagerly."""
from __future__ import annotations

import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_0811_2111_amd import xy


def replayed(make, call, out, ref_state, ref_out):
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        h = make()
        start = h.state.clone()
        call(h, out)                                       # warm-up
        h.state.copy_(start)
        h.set_sweep(0)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            call(h, out)
        for k in range(4):
            h.state.copy_(start)
            out.zero_()
            torch.randn((1 << 20,), device="cuda").sum().item()
            g.replay()
            s.synchronize()
            assert torch.equal(h.state, ref_state), k
            assert torch.equal(out.view(torch.int64), ref_out.view(torch.int64)), k


# one workgroup; several sweeps per launch, their records in one and in several
# reductions; tiles that do not divide the lattice; strips of one wave
@pytest.mark.parametrize("L,n,every", [(32, 10, 1), (256, 25, 5), (64, 300, 1), (1002, 13, 3), (1202, 5, 2), (3500, 5, 2)])
def test_sweeps_replayed(L, n, every):
    ref = xy.Lattice(L, seed=5, beta=1.05, delta=1.1)
    want = ref.sweep(n, every)
    replayed(lambda: xy.Lattice(L, seed=5, beta=1.05, delta=1.1), lambda h, o: h.sweep(n, every, out=o),
             torch.empty_like(want), ref.state, want)


@pytest.mark.parametrize("L,quad", [(32, False), (34, False), (300, False), (32, True), (96, True)])
def test_trajectories_replayed(L, quad):
    """Accepted and rejected ones in one call."""
    make = (lambda: xy.Quad(L, [1, 2, 3, 4], [0.7, 0.9, 1.1, 1.3])) if quad else (lambda: xy.Lattice(L, seed=9, beta=1.05))

    def call(h, o):
        h.hmc(3, 7, 0.1, out=o[:3])
        h.hmc(3, 7, 2.5, out=o[3:])
    ref = make()
    want = torch.empty((6, 4, 9) if quad else (6, 9), dtype=torch.float64, device="cuda")
    call(ref, want)
    assert set(xy.hmc_records(want)["accepted"].ravel().tolist()) == {0, 1}
    replayed(make, call, torch.empty_like(want), ref.state, want)
