"""The DSMC step's screen at the ends of binary32's range: speeds whose square
vanishes there, densities, cross sections and time steps that binary32 does
not hold, and particles at rest.  Channels equal to the oracle's wherever the
product that decides is an ordinary number."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, rel_err

pytestmark = pytest.mark.gpu


# speed, cross section, density, time step: their product is about 1
@pytest.mark.parametrize("dtype,speed,sigma,dens,dt", [
    (np.float32, 1e-20, 1.0, 1e20, 1.0),
    (np.float32, 1e-30, 1.0, 1e15, 1e15),
    (np.float32, 1e-35, 1e10, 1e17, 1e8),
    (np.float32, 1.0, 1e-45, 1e45, 1.0),
    (np.float32, 1.0, 1e45, 1e-45, 1.0),
    (np.float32, 1.0, 1.0, 1e50, 1e-50),
    (np.float32, 1e15, 1e-30, 1e-30, 1e45),
    (np.float64, 1e-22, 1.0, 1e22, 1.0),
    (np.float64, 1e-60, 1.0, 1e30, 1e30),
    (np.float64, 1e-60, 1.0, 1e60, 1.0),
    (np.float64, 1.0, 1e-60, 1e60, 1.0),
    (np.float64, 1.0, 1e60, 1e-60, 1.0),
    (np.float64, 1.0, 1e30, 1e20, 1e-50),
    (np.float64, 1e30, 1e-50, 1.0, 1e20),
    (np.float64, 1e60, 1e-60, 1.0, 1.0),
])
@pytest.mark.parametrize("per_cell", [False, True])
def test_screen_beyond_binary32(dtype, speed, sigma, dens, dt, per_cell):
    import torch
    from paper_2508_06771_amd import piccoll
    rng = np.random.default_rng(7)
    n, M = 5003, 10
    v = (rng.standard_normal((3, n)) * speed).astype(dtype)
    v[:, ::50] = 0.0
    cell = rng.integers(0, M, n).astype(np.int32)
    pid = rng.permutation(n).astype(np.uint32)
    top = 2.0 * float(speed) ** 2
    coef = np.zeros((4, 2, 4))
    coef[:, :, 0] = sigma * np.array([[0.3, 0.1], [0.2, 0.4], [0.0, 0.1], [0.5, 0.2]])
    coef[0, 1, 1] = 0.05 * sigma / top if np.isfinite(sigma / top) else 0.0
    # elastic and excitation from rest: no new electrons
    tab = {"breaks": np.array([0.0, 0.25, 1.0]) * top, "coef": coef, "thr": np.array([0.0, 1e300, 0.0, 1e300])}
    kw = dict(dt=dt, seed=4, step=3, pid_base=1 << 28)
    ctx = piccoll.Context(0)
    ctx.set_dsmc(tab, 1e-3)
    tv = dev(v)
    tdt = torch.float32 if dtype == np.float32 else torch.float64
    vn = torch.zeros((3, 1), dtype=tdt, device="cuda")
    pn, cn = (torch.zeros(1, dtype=torch.int32, device="cuda") for _ in range(2))
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    chan = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
    d = np.full(M, dens)
    gas = dict(n_gas=dev(d), n_meta=dev(0.5 * d)) if per_cell else dict(n_gas0=dens, n_meta0=0.5 * dens)
    ctx.dsmc_collide(tv, dev(cell), dev(pid), M, v_new=vn, pid_new=pn, cell_new=cn, count=cnt, channel_out=chan,
                     **gas, **kw)
    ctx.sync()
    ctx.close()
    r = v.astype(np.float64)
    gas = dict(n_gas=d, n_meta=0.5 * d) if per_cell else dict(ng0=dens, nm0=0.5 * dens)
    cr = oracle.dsmc(r, cell, pid, table=tab, mass_ratio=1e-3, cap=n, **gas, **kw)[0]
    assert 0.2 * n < np.count_nonzero(cr) < n
    assert np.array_equal(host(chan), cr)
    # about 20 operations in binary64 and one rounding to the stored type
    tol = 1e-5 if dtype == np.float32 else 1e-12
    assert rel_err(host(tv).astype(np.float64), r, speed) < tol
