"""Cells beyond the LDS classes, split into key segments, at the sizes where a
segment's pass can go wrong: empty, one, two, the capacity and one more than
it (the cell then takes the one-workgroup path), odd and even starts, pairs
across one and across an empty segment; and cells on both sides of the number
of segments up to which the velocities are gathered instead of copied.  The
pids are chosen by their key, so that each segment has exactly the size named.
One step with null collisions against the oracle (the bars of one step, 1e-5
in binary32, 1e-12 in binary64)."""
import numpy as np
import pytest

import oracle
from paper_2508_06771_amd import workloads
from tests.gpu_util import dev, host, rel_err

pytestmark = pytest.mark.gpu

SEED, STEP = 6, 3
# segment capacities 10,240 and 6,144, their targets 7/8 of them
SEGS = {
    "f32": (8960, [(10240, 1), (1, 10240), (10239, 2), (2, 10239), (5121, 5121), (10241, 1), (10240, 0, 10240),
                   (10239, 0, 10240), (10239, 1, 10240), (9001, 1, 9920, 9003)]),
    "f64": (5376, [(6144, 4097), (4097, 6144), (6143, 4099), (6145, 4097), (6143, 0, 6143), (6144, 1, 6144),
                   (6143, 1, 6144), (6001, 1, 5501, 5377)]),
}


def run(dtype, sizes, pid):
    import torch
    from paper_2508_06771_amd import piccoll
    rng = np.random.default_rng(21)
    sizes = np.asarray(sizes, dtype=np.int64)
    np_dtype = np.float32 if dtype == "f32" else np.float64
    v = workloads.maxwellian_beam(rng, sizes, dtype=np_dtype)
    w = workloads._finish(rng, "segments", v, sizes, np_dtype, shuffle=False, mcc=True)
    dens = rng.uniform(0.5, 2.0, w.n_cells)
    ctx = piccoll.Context(0)
    sigma0 = 30 * w.sigma0                       # about a quarter of the members scatter
    ctx.set_mcc(sigma0, 1.0, 0.0)
    tv = dev(w.v)
    kw = dict(dt=w.dt, lnL=w.lnL, seed=SEED, step=STEP)
    ctx.coulomb_collide(tv, dev(w.cell_of), dev(pid), w.n_cells, density=dev(dens), flags=piccoll.FUSE_MCC, **kw)
    ctx.sync()
    r = w.v.astype(np.float64).copy()
    oracle.step(r, w.cell_of.copy(), pid.copy(), w.n_cells, density=dens, mcc=True, sigma0=sigma0, n_neutral=1.0, **kw)
    err = rel_err(host(tv).astype(np.float64), r)
    ctx.close()
    assert err < (1e-5 if dtype == "f32" else 1e-12), err


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_segment_sizes(dtype):
    target, cells = SEGS[dtype]
    pool = np.arange(1_000_000, dtype=np.uint32)
    key = oracle.philox_fill(SEED, STEP, 0, pool)[:, 0].astype(np.uint64)
    rng = np.random.default_rng(3)
    free = np.ones(pool.size, dtype=bool)
    pids = []
    for segs in cells:
        n, s = sum(segs), len(segs)
        assert n > 10240 and -(-n // target) == s, (segs, -(-n // target))
        ids = []
        for q, m in enumerate(segs):
            own = pool[free & ((key * np.uint64(s)) >> np.uint64(32) == q)][:m]
            assert own.size == m
            free[own] = False
            ids.append(own)
        pids.append(rng.permutation(np.concatenate(ids)))
    run(dtype, [sum(c) for c in cells], np.concatenate(pids).astype(np.uint32))


def test_many_segments():
    """1,024 segments (gathered), 1,025 (copied) and 144 beside them."""
    sizes = [8960 * 1024, 8960 * 1024 + 1, 1_286_145]
    run("f32", sizes, np.random.default_rng(4).permutation(sum(sizes)).astype(np.uint32))
