"""The fused k-space kernel's routes agree with each other at every short grid
length (the oracle pins the long ones): a product of all components, which
carries both radial factors through its sums, against the same rows of
products of one kind, which apply one factor at the end (stresslets to
strains, by moments or by the kernel with three couplet grids in registers;
forces to velocities).  The same terms in another order: 1e-12 in FP64, 1e-5
in FP32."""
import numpy as np
import pytest

from gpu_common import dev, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('grid,support', [(8, 5), (12, 5), (16, 6), (24, 8), (32, 8), (48, 8),
                                          (64, 8), (96, 8), (128, 8), (192, 8), (256, 8)])
@pytest.mark.parametrize('gridding', [1, 2])
@pytest.mark.parametrize('precision,tol', [(0, 1e-12), (1, 1e-5)])
def test_one_kind_against_all_components(grid, support, gridding, precision, tol):
    import torch

    from paper_1709_06946_amd import pse
    n, L = 40, float(grid)
    if grid == 8:
        gridding = 1     # no spreading tiles, so no derivative gridding
    h = pse.PSE(n, L, grid=grid, xi=0.25, rcut=2.5, support=support, deriv_gridding=gridding,
                precision=precision)
    assert h.derived.deriv_gridding == gridding
    rng = np.random.default_rng(grid)
    x = dev(L * rng.random((n, 3)))
    q = rng.normal(size=(n, 11))
    for lo, hi in ((6, 11), (0, 3)):
        one = np.zeros_like(q)
        one[:, lo:hi] = q[:, lo:hi]
        a = torch.zeros((n, 11), dtype=torch.float64, device='cuda:0')
        h.mobility_apply(x, dev(one), a, pse.PSE_WAVE)
        if lo:
            b = torch.zeros_like(a)
            h.mobility_apply(x, dev(one), b, pse.PSE_WAVE | pse.PSE_ES_BLOCK)
            b = host(b)[:, lo:hi]
        else:
            b = torch.zeros((n, 3), dtype=torch.float64, device='cuda:0')
            h.rpy_apply(x, dev(one[:, :3]), b, pse.PSE_WAVE)
            b = host(b)
        assert rel_err(b, host(a)[:, lo:hi]) < tol
