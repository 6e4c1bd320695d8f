"""The stresslet-strain pair sum (its own kernel, alone in PSE_ES_BLOCK with
PSE_REAL) against the same rows of the whole sum, which go through the other
kernel, on lists whose rows are empty, shorter than, equal to and longer than
a group of 16 lanes; and the whole sum against the oracle's blocks below and
above the particle count from which the sums pack their moments.

Tolerances: both kernels sum the same terms of the same list, so they differ
by rounding only, 1e-13 in FP64 (up to 130 terms) and 1e-5 in FP32; against
the oracle's blocks at the list's own cutoff the table's interpolation adds
1e-9."""
import numpy as np
import pytest

from gpu_common import dev, host, rel_err

pytestmark = pytest.mark.gpu


def _cluster(m, spread, L, seed):
    """m overlapping spheres about the centre: each has m - 1 neighbours."""
    rng = np.random.default_rng(seed)
    return 0.5 * L + spread * (rng.random((m, 3)) - 0.5)


@pytest.mark.parametrize('m', [1, 2, 16, 17, 18, 33, 130])
@pytest.mark.parametrize('precision,tol', [(0, 1e-13), (1, 1e-5)])
def test_es_sum_matches_the_whole_sum(m, precision, tol):
    import torch

    from paper_1709_06946_amd import pse
    L = 30.0
    h = pse.PSE(m, L, grid=48, tol=1e-3, precision=precision)
    x = _cluster(m, 3.0, L, m)
    q = np.zeros((m, 11))
    q[:, 6:] = np.random.default_rng(1).normal(size=(m, 5))
    es = torch.zeros((m, 11), dtype=torch.float64, device='cuda:0')
    full = torch.zeros_like(es)
    h.mobility_apply(dev(x), dev(q), es, pse.PSE_REAL | pse.PSE_ES_BLOCK)
    h.mobility_apply(dev(x), dev(q), full, pse.PSE_REAL)
    assert rel_err(host(es)[:, 6:], host(full)[:, 6:]) < tol


@pytest.mark.parametrize('n', [32767, 32768])
@pytest.mark.parametrize('precision,tol', [(0, 1e-13), (1, 1e-5)])
def test_sums_on_both_sides_of_the_packed_copy(n, precision, tol):
    import torch

    from paper_1709_06946_amd import pse
    rng = np.random.default_rng(n)
    m = 32                                     # sites per side, one left out
    L = 3.0 * m
    site = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing='ij'), -1).reshape(-1, 3)[:n]
    x = 3.0 * site + rng.random((n, 3)) * 0.5
    q = rng.normal(size=(n, 11))
    h = pse.PSE(n, L, grid=128, tol=1e-3, precision=precision)
    out = torch.zeros((n, 11), dtype=torch.float64, device='cuda:0')
    h.mobility_apply(dev(x), dev(q), out, pse.PSE_REAL)
    from oracle import ewald
    rows = [0, 1, n // 2, n - 1]
    d = ewald.real_apply_rows(x, q, L, h.derived.xi, rows, rcut=h.derived.rcut)
    # the table's interpolation (1e-9) bounds the agreement in FP64
    assert rel_err(host(out)[rows], d) < max(tol, 1e-9)
