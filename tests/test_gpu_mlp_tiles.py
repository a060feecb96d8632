"""The network's gradient and optimiser step at the edges of their tiles (64
samples per workgroup, 16 groups of tiles in the reduction), binary32, against
numpy in binary64; the fused optimiser step against the gradient returned on
its own."""
import numpy as np
import pytest

from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu

# an entry of the gradient passes through about 200 binary32 roundings
TOL = 200 * 2.0 ** -24


def grad64(p, x, y):
    W1, b1, W2, b2, W3, b3 = (p[:512].reshape(8, 64), p[512:576], p[576:4672].reshape(64, 64), p[4672:4736],
                              p[4736:4800], p[4800])
    z1 = x @ W1 + b1
    a1 = np.maximum(z1, 0)
    z2 = a1 @ W2 + b2
    a2 = np.maximum(z2, 0)
    z = a2 @ W3 + b3
    loss = np.mean(np.maximum(z, 0) - z * y + np.log1p(np.exp(-np.abs(z))))
    d3 = (1 / (1 + np.exp(-z)) - y) / y.size
    d2 = d3[:, None] * W3 * (z2 > 0)
    d1 = (d2 @ W2.T) * (z1 > 0)
    return np.concatenate([(x.T @ d1).ravel(), d1.sum(0), (a1.T @ d2).ravel(), d2.sum(0), a2.T @ d3, [d3.sum()]]), loss


@pytest.mark.parametrize("batch", [1, 2, 63, 64, 65, 127, 129, 1023, 1025, 4097])
def test_gradient_and_step_at_tile_edges(batch):
    from paper_2508_06771_amd import gate, piccoll
    rng = np.random.default_rng(batch)
    p0 = gate.init_params(3).cpu().numpy()
    x = rng.standard_normal((batch, 8)).astype(np.float32)
    y = (rng.random(batch) < 0.6).astype(np.float32)
    ctx = piccoll.Context(0)
    params, tx, ty = dev(p0), dev(x), dev(y)
    g, loss = ctx.mlp_grad(params, tx, ty, bf16=False)
    ctx.sync()
    ref, lref = grad64(p0.astype(np.float64), x.astype(np.float64), y.astype(np.float64))
    got = host(g).astype(np.float64)
    assert np.linalg.norm(got - ref) < TOL * np.linalg.norm(ref)
    assert abs(host(loss)[0] - lref) < TOL * max(1.0, lref)
    m = (1e-3 * rng.standard_normal(4801)).astype(np.float32)
    v = (1e-5 * rng.random(4801)).astype(np.float32)
    tm, tv = dev(m), dev(v)
    l2 = ctx.mlp_train_step(params, tm, tv, 7, 1e-3, tx, ty, bf16=False)
    ctx.sync()
    ctx.close()
    assert host(l2)[0] == host(loss)[0]
    # the decay rates and their complements are binary32 numbers
    f = np.float32
    b1, b2, c1, c2 = (float(q) for q in (f(0.9), f(0.999), f(1) - f(0.9), f(1) - f(0.999)))
    mm, vv = b1 * m + c1 * got, b2 * v + c2 * got * got
    step = 1e-3 * (mm / (1 - 0.9 ** 7)) / (np.sqrt(vv / (1 - 0.999 ** 7)) + 1e-8)
    assert np.max(np.abs(host(tm) - mm)) < 4 * 2.0 ** -24 * np.max(np.abs(mm))
    assert np.max(np.abs(host(tv) - vv)) < 4 * 2.0 ** -24 * np.max(np.abs(vv))
    # 1 - 0.999^7 loses about 8 of its 24 bits in binary32
    assert np.max(np.abs(host(params) - (p0 - step))) < 2.0 ** -13 * np.max(np.abs(step))
