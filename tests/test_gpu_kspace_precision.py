"""The k-space columns' constants do not shift the FP32 products: the stresslet
to strain block by moments, whose columns carry -3 / sqrt 2 and 2 pi / L on
either side, against the same block by derivative gridding, whose columns are
whole numbers.  Each is compared with its own FP64 handle, by the factor that
fits best; the transforms' rounding shifts both alike.

Tolerance on the difference of the two factors: the block's spectrum is flat,
so thousands of table entries average out; the rounding noise of 1.5e-7 over
1000 strains leaves 5e-9, and the transforms' own shift (6e-8 each way)
differs between the two fields by about a tenth.  4e-8 covers both; columns
rounded with their constants are off by 4e-8 to 1.3e-7, by box."""
import numpy as np
import pytest

from gpu_common import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('L', [20.0, 24.0, 30.0, 33.3, 41.7])
def test_columns_are_not_shifted(L):
    import torch

    from paper_1709_06946_amd import pse
    n, grid = 200, 48
    rng = np.random.default_rng(5)
    x, q = dev(L * rng.random((n, 3))), dev(rng.normal(size=(n, 11)))
    factor = []
    for gridding in (1, 2):
        e = []
        for precision in (0, 1):
            h = pse.PSE(n, L, grid=grid, tol=1e-3, precision=precision, deriv_gridding=gridding)
            out = torch.zeros((n, 11), dtype=torch.float64, device='cuda:0')
            h.mobility_apply(x, q, out, pse.PSE_WAVE | pse.PSE_ES_BLOCK)
            e.append(host(out)[:, 6:])
        factor.append((e[1] * e[0]).sum() / (e[0] ** 2).sum())
    print(L, factor[0] - 1, factor[1] - 1)
    assert abs(factor[0] - factor[1]) < 4e-8
