"""Work lists around the number of workgroups and queues that share them: lists
shorter than the queues, one cell more or fewer than the takers, and many
cells per queue, in every size class; each cell is collided exactly once (the
step equals the oracle's)."""
import numpy as np
import pytest

import oracle
from paper_2508_06771_amd import workloads
from tests.gpu_util import dev, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tol", [(np.float32, 1e-5), (np.float64, 1e-12)])
@pytest.mark.parametrize("cells,size", [(1, 2), (15, 40), (16, 40), (17, 40), (127, 30), (2049, 3), (9000, 9),
                                        (1025, 520), (4200, 514), (513, 2100), (15, 4100), (257, 4101),
                                        (15, 10300), (40, 10300)])
def test_every_cell_once(cells, size, dtype, tol):
    import torch
    from paper_2508_06771_amd import piccoll
    rng = np.random.default_rng(cells)
    # ragged, the first cell of the largest size; an empty one and a single member
    sizes = np.maximum(size - rng.integers(0, 3, cells), 0)
    sizes[0] = size
    if cells > 10:
        sizes[3], sizes[7] = 0, 1
    v = workloads.maxwellian_beam(rng, sizes.astype(np.int64), dtype=dtype)
    w = workloads._finish(rng, "queues", v, sizes.astype(np.int64), dtype, shuffle=False, mcc=True)
    ctx = piccoll.Context(0)
    ctx.set_mcc(w.sigma0, w.n_neutral, 0.0)
    tv, tc, tp = dev(w.v), dev(w.cell_of), dev(w.pid)
    for schedule in (0, 1):
        ctx.set_schedule(torch.float32 if dtype == np.float32 else torch.float64, schedule)
        x = tv.clone()
        ctx.coulomb_collide(x, tc, tp, w.n_cells, dt=w.dt, lnL=w.lnL, seed=5, step=2, flags=piccoll.FUSE_MCC)
        ctx.sync()
        if schedule == 0:
            first = x
        else:
            assert torch.equal(first, x)
    ctx.close()
    r = w.v.astype(np.float64).copy()
    oracle.step(r, w.cell_of.copy(), w.pid.copy(), w.n_cells, dt=w.dt, lnL=w.lnL, seed=5, step=2, mcc=True,
                sigma0=w.sigma0, n_neutral=w.n_neutral)
    assert rel_err(host(first).astype(np.float64), r) < tol
