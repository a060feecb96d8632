"""The binary32 correction in cells of the largest LDS class runs on one kernel
where the electrons fill at most a cell per workgroup and on another beyond: a
cell's velocities are the same bit for bit on both, and the oracle's."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [4097, 6501, 10047, 10240])
def test_same_velocities_alone_and_among_many(size):
    import torch
    from paper_2508_06771_amd import piccoll
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(size)
    cells = cu + 3                      # the list may hold more than a cell per workgroup
    n = cells * size
    v = (rng.normal(size=(3, n)) * np.array([[1.0], [1.0], [1.4]])).astype(np.float32)
    pid = rng.permutation(n).astype(np.uint32)
    cell = np.repeat(np.arange(cells, dtype=np.int32), size)
    kw = dict(dt=0.01, lnL=10.0, seed=6, step=3)
    out = []
    for part in (slice(0, n), slice(0, 2 * size)):
        ctx = piccoll.Context(0)
        tv = dev(np.ascontiguousarray(v[:, part]))
        ctx.coulomb_collide(tv, dev(cell[part].copy()), dev(pid[part].copy()), (part.stop - part.start) // size,
                            flags=piccoll.CONSERVE_FIX, **kw)
        ctx.sync()
        ctx.close()
        out.append(host(tv))
    assert np.array_equal(out[0][:, :2 * size], out[1])
    ref = v[:, :2 * size].astype(np.float64)
    oracle.step(ref, cell[:2 * size].copy(), pid[:2 * size].copy(), 2, conserve=True, **kw)
    assert rel_err(out[1].astype(np.float64), ref) < 1e-5      # the binary32 bar of one step
