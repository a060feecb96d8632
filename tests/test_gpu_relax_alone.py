"""A cell's relaxation label depends on the cell alone: bit for bit the same
with no other cell in the call as among many, whose number decides how the
replicas are dealt to workgroups."""
import numpy as np
import pytest

from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("replicas", [1, 3, 8, 11])
def test_label_alone_and_in_company(dtype, replicas):
    from paper_2508_06771_amd import piccoll
    rng = np.random.default_rng(9)
    probes = [2, 5, 300, 512, 513, 2048, 2049, 6500, 10240]
    sizes = np.array(probes + [40] * 3000 + [2100] * 300)
    cs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(cs[-1])
    v = rng.standard_normal((3, n)) * np.array([[1.0], [1.1], [1.4]])
    v = v.astype(np.float32) if dtype == "f32" else v
    pid = rng.permutation(n).astype(np.uint32)
    kw = dict(dt=1e-3, lnL=10.0, seed=3, step=4, replicas=replicas)
    ctx = piccoll.Context(0)
    all_r = host(ctx.relaxation(dev(v), dev(cs), dev(pid), **kw))
    for j in range(len(probes)):
        part = slice(cs[j], cs[j + 1])
        alone = np.array([0, sizes[j]], np.int32)
        r = host(ctx.relaxation(dev(np.ascontiguousarray(v[:, part])), dev(alone), dev(pid[part].copy()), **kw))
        assert r[0] == all_r[j], (sizes[j], r[0], all_r[j])
    ctx.sync()
    ctx.close()
