"""A synchronous Lanczos solve stops at the first iteration that meets the
tolerance (or exhausts the Krylov space), whatever the handle solved before:
its samples and counts are those of a new handle, bit for bit.

After a solve of many iterations the host first looks late; the easier solves
here end at least three iterations before that look.  One, few and many
launches per step (vectors of 2048 and 2^18 numbers lie between the sizes)."""
import numpy as np
import pytest

from gpu_common import dev, host

pytestmark = pytest.mark.gpu


def _sites(n, spacing, jitter, rng):
    m = int(np.ceil(n ** (1 / 3) - 1e-9))
    site = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing='ij'), -1).reshape(-1, 3)[:n]
    return spacing * site + jitter * rng.random((n, 3))


@pytest.mark.parametrize('n,grid', [(125, 64), (1000, 128), (24000, 192)])
@pytest.mark.parametrize('precision', [0, 1])
@pytest.mark.parametrize('easy', ['sparse', 'isolated'])
def test_easier_solves_match_a_new_handle(n, grid, precision, easy):
    import torch

    from paper_1709_06946_amd import pse
    m = int(np.ceil(n ** (1 / 3) - 1e-9))
    L = 11.0 * m
    rng = np.random.default_rng(n)
    hard = _sites(n, 2.02, 0.01, rng)                      # a touching clump
    x = _sites(n, 11.0, 5.0 if easy == 'sparse' else 0.0, rng)
    psi = dev(rng.normal(size=(n, 11)))

    def sample(h, pos):
        out = torch.zeros((n, 11), dtype=torch.float64, device='cuda:0')
        rc, st = h.brownian_sample(dev(pos), psi, out_real=out)
        assert rc == 0
        return host(out), st

    def handle():
        return pse.PSE(n, L, grid=grid, tol=1e-3, precision=precision, lanczos_tol=1e-4)

    want, st = sample(handle(), x)
    old = handle()
    _, before = sample(old, hard)
    assert before['lanczos_iters'] >= st['lanczos_iters'] + 4
    for _ in range(2):
        got, now = sample(old, x)
        assert now == st
        assert np.array_equal(got, want)
        sample(old, hard)
