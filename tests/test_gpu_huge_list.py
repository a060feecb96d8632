"""More cells beyond the LDS classes than workgroups that take them, in each
form of their kernel (weights, Nanbu's operator, the triplet, the correction):
every one is collided once, bit for bit as in calls of 25 cells; three cells
(fewer than queue lines) against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, rel_err

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-5, "f64": 1e-12}     # one step from the same state, as for the smaller classes
KW = dict(dt=0.01, lnL=10.0, seed=6, step=3)
SIZE = {"f32": 10250, "f64": 6170}


def population(cells, size):
    rng = np.random.default_rng(cells)
    counts = size + rng.integers(0, 4, cells)
    cs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    n = int(cs[-1])
    v = rng.normal(size=(3, n)) * np.array([[1.0], [1.0], [1.4]])
    return v, rng.permutation(n).astype(np.uint32), rng.choice([0.5, 1.0, 2.0], n), cs


def collide(ctx, op, v, pid, w, cs, tdt):
    from paper_2508_06771_amd import piccoll
    tv = dev(np.ascontiguousarray(v), tdt)
    if op == "fix":
        cell = np.repeat(np.arange(cs.size - 1, dtype=np.int32), np.diff(cs))
        ctx.coulomb_collide(tv, dev(cell), dev(pid.copy()), cs.size - 1, flags=piccoll.CONSERVE_FIX, **KW)
        ctx.conserve_reset()
    elif op == "weighted":
        ctx.weighted(tv, dev(w.copy(), tdt), dev(pid.copy()), dev(cs), **KW)
    elif op == "nanbu":
        ctx.nanbu(tv, dev(pid.copy()), dev(cs), **KW)
    else:
        ctx.triplet(tv, dev(pid.copy()), dev(cs), **KW)
    ctx.sync()
    return host(tv)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("op", ["weighted", "nanbu", "triplet", "fix"])
def test_more_cells_than_workgroups(op, dtype):
    import torch
    from paper_2508_06771_amd import piccoll
    v, pid, w, cs = population(300, SIZE[dtype])
    tdt = torch.float32 if dtype == "f32" else torch.float64
    ctx = piccoll.Context(0)
    got = collide(ctx, op, v, pid, w, cs, tdt)
    for a in range(0, 300, 25):
        part = slice(cs[a], cs[a + 25])
        ref = collide(ctx, op, v[:, part], pid[part], w[part], cs[a:a + 26] - cs[a], tdt)
        assert np.array_equal(got[:, part], ref), a
    ctx.close()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("op", ["weighted", "nanbu", "triplet", "fix"])
def test_three_cells_against_the_oracle(op, dtype):
    import torch
    from paper_2508_06771_amd import piccoll
    v, pid, w, cs = population(3, SIZE[dtype])
    tdt = torch.float32 if dtype == "f32" else torch.float64
    ctx = piccoll.Context(0)
    got = collide(ctx, op, v, pid, w, cs, tdt).astype(np.float64)
    ctx.close()
    ref = host(dev(v, tdt)).astype(np.float64)
    if op == "fix":
        cell = np.repeat(np.arange(3, dtype=np.int32), np.diff(cs))
        oracle.step(ref, cell, pid.copy(), 3, conserve=True, **KW)
    elif op == "weighted":
        oracle.step_weighted(ref, w, cs, pid, 0.01, 10.0, 6, 3)
    elif op == "nanbu":
        oracle.nanbu(ref, cs, pid, 0.01, 10.0, 6, 3, None)
    else:
        oracle.step_triplet(ref, cs, pid, 0.01, 10.0, 6, 3)
    assert rel_err(got, ref) < TOL[dtype]
