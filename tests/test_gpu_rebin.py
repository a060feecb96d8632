"""Re-binning of unsorted storage: the counting sort moves cell ids, pids and
velocities together and stably, checked against numpy's stable argsort at the
edges of its tiles (4,096 elements), of its workgroups' runs (512 workgroups,
so several tiles each beyond 2,097,152 elements) and of its digits."""
import numpy as np
import pytest

from tests.gpu_util import dev, host, host_u32

pytestmark = pytest.mark.gpu

# a step this weak turns no velocity: what comes back is what was moved
LNL = 1e-300


@pytest.fixture(scope="module")
def ctx():
    from paper_2508_06771_amd import piccoll
    c = piccoll.Context(0)
    yield c
    c.sync()
    c.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,M", [(2, 2), (63, 5), (4095, 3), (4096, 256), (4097, 257), (8193, 4096), (70001, 65536),
                                 (100003, 70000), (300000, 2_000_000), (2097152, 1000), (2097153, 511),
                                 (2500001, 40000)])
@pytest.mark.parametrize("order", ["shuffled", "neighbours", "reversed"])
def test_rebin_moves_stably(ctx, n, M, dtype, order):
    rng = np.random.default_rng(n + M)
    cell = np.sort(rng.integers(0, M, n)).astype(np.int32)
    if order == "shuffled":
        cell = rng.permutation(cell)
    elif order == "reversed":
        cell = cell[::-1].copy()
    else:
        hop = rng.random(n) < 0.05
        cell = np.where(hop, (cell + rng.choice([-1, 1], n)) % M, cell).astype(np.int32)
        cell[0], cell[-1] = M - 1, 0
    v = rng.standard_normal((3, n)).astype(dtype)
    pid = rng.permutation(n).astype(np.uint32)
    tv, tc, tp = dev(v), dev(cell), dev(pid)
    ctx.coulomb_collide(tv, tc, tp, M, dt=1e-3, lnL=LNL, seed=1, step=0)
    ctx.sync()
    o = np.argsort(cell, kind="stable")
    assert np.array_equal(host(tc), cell[o])
    assert np.array_equal(host_u32(tp), pid[o])
    assert np.array_equal(host(tv), v[:, o])


@pytest.mark.parametrize("n,M,skip", [(5000, 300, 1), (70000, 4000, 3), (2200000, 4096, 2)])
def test_bin_cells_of_an_unaligned_view(ctx, n, M, skip):
    rng = np.random.default_rng(n)
    cell = rng.integers(0, M, n + skip).astype(np.int32)
    cs, order = ctx.bin_cells(dev(cell)[skip:], M)
    ctx.sync()
    cell = cell[skip:]
    assert np.array_equal(host(order), np.argsort(cell, kind="stable"))
    assert np.array_equal(host(cs), np.concatenate([[0], np.cumsum(np.bincount(cell, minlength=M))]))
