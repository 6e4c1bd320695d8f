"""Interpolation against the plain sum over each particle's stencil: every
support (its own instance or the next one's), component counts that fill an
instance and that do not, grids with spreading tiles and without, particles at
the box's faces.  Tolerances as for the other interpolations: 1e-12 in FP64,
2e-6 of the single precision grids."""
import numpy as np
import pytest

from gpu_common import dev, host
from test_gpu_kernels import _interp_ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('grid,support', [(8, 2), (8, 6), (12, 3), (16, 4), (24, 16), (32, 5),
                                          (48, 7), (48, 9), (64, 10), (32, 11), (48, 13),
                                          (48, 16)])
@pytest.mark.parametrize('ncomp', [1, 4, 6, 11])
@pytest.mark.parametrize('precision,tol', [(0, 1e-12), (1, 2e-6)])
def test_interpolation_at_every_support(grid, support, ncomp, precision, tol):
    import torch

    from paper_1709_06946_amd import pse
    n, L = 61, float(grid)
    h = pse.PSE(n, L, grid=grid, xi=0.25, rcut=2.5, support=support, precision=precision)
    assert h.derived.support == support
    rng = np.random.default_rng(grid + support)
    x = L * rng.random((n, 3))
    x[:3] = [[0.0, 0.0, 0.0], [np.nextafter(L, 0.0)] * 3, [0.5, 1.0, L - 0.5]]
    field = rng.normal(size=(ncomp, grid, grid, grid))
    out = torch.zeros((n, ncomp), dtype=torch.float64, device='cuda:0')
    h.interpolate(dev(x), dev(field), out)
    ref = _interp_ref(h, x, field)
    assert np.abs(host(out) - ref).max() < tol * np.abs(ref).max()
