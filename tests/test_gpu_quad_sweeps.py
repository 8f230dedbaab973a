"""The schedules a quad's sweeps take where no tile was asked for (the whole quad in
four workgroups, passes of several sweeps, single sweeps of the lattices apart)
against the one-kernel sweep that a chosen tile takes."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_0811_2111_amd import xy

SEEDS, BETAS, DELTAS = [3, 4, 1 << 40, 6], [0.7, 1.0, 1.2, 2.0], [1.0, 1.2, 0.8, 0.5]


def pair(L):
    a, b = xy.Quad(L, SEEDS, BETAS, DELTAS), xy.Quad(L, SEEDS, BETAS, DELTAS)
    b.set_tile(32, 16)
    return a, b


# 32: one workgroup a replica; 64: records fill the workspace after two sweeps; 96,
# 160: uneven regions; 384, 416: two and four pairs a thread; 576, 608: the last side
# in passes, the first in tiles (128-wide, the last of 96 columns); 1024: whole
# 256-wide ones; 2976: past the last-level cache
@pytest.mark.parametrize("L", [32, 64, 96, 160, 384, 416, 576, 608, 1024, 2976])
def test_quad_schedules_match_one_kernel(L):
    a, b = pair(L)
    for n, every in [(1, 1), (2, 1), (2, 0), (3, 1), (10, 1), (10, 10), (13, 3)]:
        oa, ob = a.sweep(n, every), b.sweep(n, every)
        assert torch.equal(a.state, b.state) and a.sweep_count == b.sweep_count, (n, every)
        if every:
            for r in range(4):
                ra, rb = xy.records(oa[:, r]), xy.records(ob[:, r])
                assert np.array_equal(ra["sweep"], rb["sweep"]) and np.array_equal(ra["n_accept"], rb["n_accept"])
                for f in ("cx", "cy", "ix", "iy", "mx", "my"):
                    # the same FP32 terms (a pair of sites each, below 8) in FP64 sums of another order
                    np.testing.assert_allclose(ra[f], rb[f], rtol=0, atol=2.0 ** -52 * 8 * L * L)


def test_quad_graph_replay():
    """Captured passes replayed with the state put back in between."""
    for L in (96, 544, 864):
        a, b = pair(L)
        out = torch.empty((3, 4, 8), dtype=torch.float64, device="cuda")
        start = a.state.clone()
        ref = b.sweep(9, 3)
        s = torch.cuda.Stream()
        q = None
        with torch.cuda.stream(s):
            q = xy.Quad(L, SEEDS, BETAS, DELTAS)
            q.sweep(9, 3, out=out)
            q.state.copy_(start)
            q.set_sweep(0)
            s.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                q.sweep(9, 3, out=out)
            for _ in range(3):
                q.state.copy_(start)
                out.zero_()
                g.replay()
                s.synchronize()
                assert torch.equal(q.state, b.state)
                assert torch.equal(out.view(torch.int64)[..., :2], ref.view(torch.int64)[..., :2])


@pytest.mark.parametrize("L", [96, 544, 864])
def test_quad_injected_failure(L):
    n = 9
    _, ref = pair(L)
    ref.sweep(n)
    for after in (0, 1, 2, 4, 6):
        q = xy.Quad(L, SEEDS, BETAS, DELTAS)
        xy.xy_test_inject_failure(after)
        try:
            q.sweep(n, 3)
        except xy.XYError:
            pass
        finally:
            xy.xy_test_inject_failure(-1)
        q.sweep(n - q.sweep_count)
        assert torch.equal(q.state, ref.state) and q.sweep_count == n, after
