"""The widest stencil (support 16, which a tolerance of 1e-9 asks for): no
spreading tile holds it, so such handles spread by atomics and interpolate
without weight rows.

Tolerances: spreading as the other spreading tests (1e-12, and 2e-6 of single
precision grids); products within the tolerance their handle was made for
(1e-5; the 1e-9 handle is held to 1e-7, above the radial table's 1e-9 and the
Ewald sums' own)."""
import numpy as np
import pytest

from gpu_common import block_errors, dev, host
from oracle import ewald
from test_gpu_kernels import _spread_ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('grid', [24, 48, 64])
@pytest.mark.parametrize('precision,tol', [(0, 1e-12), (1, 2e-6)])
def test_spreading(grid, precision, tol):
    import torch

    from paper_1709_06946_amd import pse
    n, L = 61, float(grid)
    h = pse.PSE(n, L, grid=grid, xi=0.25, rcut=2.5, support=16, precision=precision)
    rng = np.random.default_rng(grid)
    x = L * rng.random((n, 3))
    x[:2] = [[0.0, 0.0, 0.0], [np.nextafter(L, 0.0)] * 3]
    q = rng.normal(size=(n, 11))
    g = torch.full((11, grid, grid, grid), 9.0, dtype=torch.float64, device='cuda:0')
    h.spread(dev(x), dev(q), g)
    ref = _spread_ref(h, x, q)
    assert np.abs(host(g) - ref).max() < tol * np.abs(ref).max()


@pytest.mark.parametrize('L,grid,tol,support,bound', [(20.0, 48, 1e-5, 16, 1e-5),
                                                      (24.0, 64, 1e-9, 0, 1e-7)])
def test_product_and_step(L, grid, tol, support, bound):
    import torch

    from paper_1709_06946_amd import pse
    n = 20
    rng = np.random.default_rng(3)
    site = np.stack(np.meshgrid(*[np.arange(3)] * 3, indexing='ij'), -1).reshape(-1, 3)[:n]
    x = site * (L / 3) + rng.random((n, 3)) * (L / 3 - 2.5)
    q = rng.normal(size=(n, 11))
    h = pse.PSE(n, L, grid=grid, tol=tol, support=support)
    assert h.derived.support == 16
    out = torch.zeros((n, 11), dtype=torch.float64, device='cuda:0')
    h.mobility_apply(dev(x), dev(q), out)
    ref = (ewald.grand_dense(x, L, h.derived.xi) @ q.reshape(-1)).reshape(n, 11)
    err = block_errors(host(out), ref)
    print(err)
    assert max(err.values()) < bound
    xt = dev(x)
    rc, st = h.constrained_step(xt, dev(q[:, :6].copy()), 1e-3, seed=1)
    assert rc == 0 and st['converged'] == 1 and np.isfinite(host(xt)).all()
