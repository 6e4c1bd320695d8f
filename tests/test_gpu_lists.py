"""The lists that a position update builds, and spreading from them: the
binnings of one workgroup and of several launches give the same sums; a pair
list longer than its capacity makes the call start over, with the same results
as on a handle that has grown already; the tile gather at the edges of its
tiles (4^3 and 8^3 points, tile lattices that do and do not divide by four, the
shortest and longest stencils, tiles with more particles than one chunk).

Tolerances: the same terms in another order, 1e-12 (FP64) and 2e-6 of the
single precision grids (as the other spreading tests); the wave-space product
is symmetric in exact arithmetic, its two halves differing by the rounding of
spreading, transforms and interpolation: 1e-12 and 1e-5."""
import numpy as np
import pytest

from gpu_common import dev, host, rel_err
from test_gpu_kernels import _spread_ref

pytestmark = pytest.mark.gpu


def _lattice(n, spacing, rng):
    m = int(np.ceil(n ** (1 / 3) - 1e-9))
    site = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing='ij'), -1).reshape(-1, 3)[:n]
    return spacing * site + 0.4 * rng.random((n, 3))


@pytest.mark.parametrize('precision,tol', [(0, 1e-12), (1, 1e-5)])
def test_bins_on_both_sides_of_one_workgroup(precision, tol):
    import torch

    from paper_1709_06946_amd import pse
    rng = np.random.default_rng(7)
    n, L = 4096, 50.0
    x = _lattice(n + 1, 2.9, rng)
    q = rng.normal(size=(n + 1, 11))
    q[n] = 0.0                     # the sphere that only the second handle has
    p = np.concatenate([rng.permutation(n), [n]])
    out = []
    for k in (n, n + 1):
        h = pse.PSE(k, L, grid=64, tol=1e-3, precision=precision)
        t = torch.zeros((k, 11), dtype=torch.float64, device='cuda:0')
        h.mobility_apply(dev(x[p[:k]]), dev(q[p[:k]]), t)
        out.append(host(t))
    assert rel_err(out[1][:n], out[0]) < tol


@pytest.mark.parametrize('precision', [0, 1])
def test_a_step_whose_pair_list_grows(precision):
    import torch

    from paper_1709_06946_amd import pse
    rng = np.random.default_rng(11)
    n, L = 216, 70.0
    # a clump: over a hundred neighbours each, against 2 at the mean density, of
    # which the list has room for twice as many at first
    x = 20.0 + _lattice(n, 2.5, rng)
    FL = rng.normal(size=(n, 6))
    h = pse.PSE(n, L, grid=64, tol=1e-3, precision=precision)
    got = []
    for _ in range(2):
        xt = dev(x)
        o = [torch.zeros((n, k), dtype=torch.float64, device='cuda:0') for k in (5, 3)]
        h.constrained_step(xt, dev(FL), 1e-3, seed=3, step=2, stresslet=o[0], velocity=o[1])
        got.append([host(t) for t in (xt, *o)])
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize('grid,support', [(12, 2), (12, 7), (16, 6), (24, 15), (48, 14), (64, 5)])
@pytest.mark.parametrize('ncomp', [1, 6, 7, 11])
@pytest.mark.parametrize('precision,tol', [(0, 1e-12), (1, 2e-6)])
def test_spread_at_the_edges_of_tiles(grid, support, ncomp, precision, tol):
    import torch

    from paper_1709_06946_amd import pse
    n, L = 61, float(grid)
    h = pse.PSE(n, L, grid=grid, xi=0.25, rcut=2.5, support=support, precision=precision)
    assert h.derived.support == support
    rng = np.random.default_rng(grid + support)
    x = L * rng.random((n, 3))
    x[:40] = (x[:40] * 3.0 / L) % L          # a crowd at the box's corner
    x[40:43] = [[0.0, 0.0, 0.0], [np.nextafter(L, 0.0)] * 3, [0.5, 1.0, 1.5]]
    q = rng.normal(size=(n, ncomp))
    g = torch.full((ncomp, grid, grid, grid), 9.0, dtype=torch.float64, device='cuda:0')
    h.spread(dev(x), dev(q), g)
    ref = _spread_ref(h, x, q)
    assert np.abs(host(g) - ref).max() < tol * np.abs(ref).max()


@pytest.mark.parametrize('grid,support', [(12, 5), (16, 6), (24, 10), (48, 8), (64, 5)])
@pytest.mark.parametrize('block', [0, 4])
@pytest.mark.parametrize('precision,tol', [(0, 1e-12), (1, 1e-5)])
def test_gradient_spreading_is_the_transpose_of_interpolation(grid, support, block, precision,
                                                              tol):
    import torch

    from paper_1709_06946_amd import pse
    n, L = 61, float(grid)
    h = pse.PSE(n, L, grid=grid, xi=0.25, rcut=2.5, support=support, deriv_gridding=2,
                precision=precision)
    rng = np.random.default_rng(grid)
    x = L * rng.random((n, 3))
    x[:40] = x[:40] * 3.0 / L
    v = rng.normal(size=(2, n, 11))
    if block:
        v[:, :, :6] = 0.0
    Mv = []
    for q in v:
        t = torch.zeros((n, 11), dtype=torch.float64, device='cuda:0')
        h.mobility_apply(dev(x), dev(q), t, pse.PSE_WAVE | block)
        Mv.append(host(t))
    gap = abs((v[0] * Mv[1]).sum() - (v[1] * Mv[0]).sum())
    assert gap < tol * np.linalg.norm(v[0]) * np.linalg.norm(Mv[1])


@pytest.mark.parametrize('grid,support', [(24, 5), (32, 8), (48, 9), (48, 13), (64, 14), (32, 16)])
@pytest.mark.parametrize('ncomp', [1, 5, 11])
@pytest.mark.parametrize('precision,tol', [(0, 1e-12), (1, 2e-6)])
def test_spread_and_interpolate_on_a_deformed_lattice(grid, support, ncomp, precision, tol):
    import torch

    from paper_1709_06946_amd import pse
    n, L = 61, float(grid)
    A = np.array([[1.0, 0.3, -0.1], [0.0, 1.0, 0.2], [0.0, 0.0, 1.0]])
    h = pse.PSE(n, L, grid=grid, xi=0.25, rcut=2.2, support=support, precision=precision,
                deform=A.tolist())
    d = h.derived
    assert d.support == support
    rng = np.random.default_rng(grid + support)
    u = L * rng.random((n, 3))                  # lattice coordinates
    u[:40] = u[:40] * 3.0 / L
    u[40:42] = [[0.0, 0.0, 0.0], [0.5, 1.0, L - 0.5]]
    q = rng.normal(size=(n, ncomp))
    P, hh = support, d.h
    f = u / hh
    start = (np.floor(f + 0.5).astype(int) - (P - 1) // 2 if P % 2
             else np.floor(f).astype(int) - P // 2 + 1)
    idx = start[:, :, None] + np.arange(P)
    off = idx * hh - u[:, :, None]
    kcoef = 2 * d.xi**2 / d.eta_s
    kn = np.sqrt(2 * d.xi**2 / (np.pi * d.eta_s))
    field = rng.normal(size=(ncomp, grid, grid, grid))
    ref, val = np.zeros_like(field), np.zeros((n, ncomp))
    for p in range(n):
        dd = np.stack(np.meshgrid(off[p, 2], off[p, 1], off[p, 0], indexing='ij')[::-1], -1)
        W = kn**3 * np.exp(-kcoef * ((dd @ A.T) ** 2).sum(-1))
        iz, iy, ix = np.ix_(*(idx[p, a] % grid for a in (2, 1, 0)))
        for c in range(ncomp):
            np.add.at(ref[c], (iz, iy, ix), W * q[p, c])
        val[p] = (field[:, iz, iy, ix] * W).sum(axis=(1, 2, 3))
    x = dev(u @ A.T)
    g = torch.full(field.shape, 9.0, dtype=torch.float64, device='cuda:0')
    h.spread(x, dev(q), g)
    assert np.abs(host(g) - ref).max() < tol * np.abs(ref).max()
    out = torch.zeros((n, ncomp), dtype=torch.float64, device='cuda:0')
    h.interpolate(x, dev(field), out)
    assert np.abs(host(out) - val).max() < tol * np.abs(val).max()
