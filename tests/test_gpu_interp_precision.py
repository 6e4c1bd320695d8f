"""Interpolation from FP32 grids forms weights, products and sums in FP64: a
mixed handle gives the FP64 handle's values on a field that single precision
holds exactly.  The same numbers are summed in the same order, so 1e-14 of the
largest value leaves a few roundings' room; weights rounded to single
precision miss it by a factor of a million."""
import numpy as np
import pytest

from gpu_common import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('support,gridding', [(4, 1), (5, 1), (7, 1), (8, 1), (10, 1), (12, 1),
                                              (15, 1), (5, 2), (7, 2), (8, 2), (10, 2)])
def test_mixed_interpolation_rounds_nothing_but_the_grid(support, gridding):
    import torch

    from paper_1709_06946_amd import pse
    n, grid = 500, 48
    L = float(grid)
    rng = np.random.default_rng(support)
    x = dev(L * rng.random((n, 3)))
    field = rng.normal(size=(5, grid, grid, grid)) + 3.0
    field = dev(field.astype(np.float32).astype(np.float64))
    got = []
    for precision in (0, 1):
        h = pse.PSE(n, L, grid=grid, xi=0.25, rcut=2.5, support=support,
                    deriv_gridding=gridding, precision=precision)
        out = torch.zeros((n, 5), dtype=torch.float64, device='cuda:0')
        h.interpolate(x, field, out)
        got.append(host(out))
    assert np.abs(got[1] - got[0]).max() < 1e-14 * np.abs(got[0]).max()
