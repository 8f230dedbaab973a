"""One leap-frog step per launch on batches and on the four-replica texel against the
single lattices' trajectories, at sides that are no multiple of the rows or columns a
workgroup takes, and against passes of several steps."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_0811_2111_amd import xy


# one and two column blocks (J = L / 4 below and above 256), a single step and several
@pytest.mark.parametrize("Ls", [[4, 36, 100], [1020, 1028, 64], [2052, 500]])
def test_batch_of_single_steps(Ls):
    n = len(Ls)
    for n_md, steps in ((6, 1), (1, 7)):
        b = xy.Batch(Ls, range(n), [1.0 + 0.1 * i for i in range(n)], [1.0] * n)
        b.set_hmc_steps_per_pass(steps)
        rec = xy.hmc_records(b.hmc(3, n_md, 0.1))
        for i, L in enumerate(Ls):
            lat = xy.Lattice(L, seed=i, beta=1.0 + 0.1 * i)
            srec = xy.hmc_records(lat.hmc(3, n_md, 0.1))
            assert srec.tobytes() == rec[i].tobytes() and torch.equal(b.lattice_state(i), lat.state), (L, n_md)


@pytest.mark.parametrize("L", [32, 96, 1056])
def test_quad_of_single_steps(L):
    args = ([1, 2, 3, 4], [0.7, 0.9, 1.1, 1.3])
    for n_md in (1, 4, 5):
        a, b = xy.Quad(L, *args), xy.Quad(L, *args)
        a.set_hmc_steps_per_pass(1)
        ra, rb = xy.hmc_records(a.hmc(2, n_md, 0.2)), xy.hmc_records(b.hmc(2, n_md, 0.2))
        assert torch.equal(a.state, b.state) and np.array_equal(ra["accepted"], rb["accepted"]), n_md
        assert ra.tobytes() == rb.tobytes()                # the same sums in the same order
