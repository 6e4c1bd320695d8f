"""The stage profiler counts the bytes of the pair sums on handles created
asynchronous too, whose list length the host never reads."""
import numpy as np
import pytest

from gpu_common import dev, packing

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('precision', [0, 1])
def test_pair_sums_have_bytes(precision):
    import torch

    from paper_1709_06946_amd import pse
    n = 300
    x, L = packing(n, 0.1, 77)
    got = []
    for async_calls in (0, 1):
        h = pse.PSE(n, L, grid=32, tol=1e-3, precision=precision, async_calls=async_calls)
        xt = dev(x)
        h.constrained_step(xt, None, 1e-3, seed=1)
        h.profile(True)
        h.constrained_step(xt, None, 1e-3, seed=1, step=1)
        torch.cuda.synchronize()
        real = h.profile_read()['real']
        got.append(real['alg_bytes'] / real['launches'])
        h.profile(False)
    # an asynchronous list keeps twice the capacity of a uniform suspension's
    assert got[0] / 4 < got[1] < 16 * got[0]
