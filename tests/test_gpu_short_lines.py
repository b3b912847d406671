"""The fused x-y passes of short lines (FFT lengths 24, 32, 48, 64 along x and y)
against the oracle's direct FP64 rows: box products and solves on grids that
mix the lengths, with ragged extents (planes shorter than a batch of lines,
columns that end inside one, z blocks with padding rows).

Bars: FP64 products 1e-12 of the largest entry, FP32 products 5e-6 (the
operator's bars elsewhere); solved systems: the oracle's residual of the
returned w is at most twice the tolerance (the solver's own test plus FP64
rounding)."""

import numpy as np
import pytest

from oracle import vie_dense as vd
from synth import Grid

pytestmark = pytest.mark.gpu
K0 = 2 * np.pi

GRIDS = [(11, 30, 5), (24, 13, 9), (32, 32, 20), (17, 9, 16), (9, 25, 33), (16, 16, 16)]


@pytest.fixture(scope="module")
def V():
    import torch

    assert torch.cuda.is_available()
    from paper_2508_16471_amd import vie

    vie.lib()
    return vie


def _body(n):
    rng = np.random.default_rng(sum(n))
    g = Grid.centred(n, 0.05)
    return rng, g, np.where(rng.random(n[::-1]) < 0.6, rng.uniform(1.2, 2.0, n[::-1]), 1.0)


@pytest.mark.parametrize("n", GRIDS)
def test_box_products_match_oracle_rows(V, n):
    rng, g, eps = _body(n)
    x = rng.standard_normal((3, 3) + eps.shape) + 1j * rng.standard_normal((3, 3) + eps.shape)
    pos = vd.voxel_centres(g.n, g.h, g.origin)
    rows = rng.choice(eps.size, 24, replace=False)
    # a second body of the same grid: the product must take this body's chi
    ctx = V.vie_setup([(np.full(eps.shape, 1.5), g.h, g.origin), (eps, g.h, g.origin)],
                      V.make_options(K0))
    try:
        assert all(p in (24, 32, 48, 64) for p in V.vie_grid(ctx, 1)[1][:2])
        for prec, bar in ((V.VIE_FP64, 1e-12), (V.VIE_MIXED, 5e-6)):
            y = V.vie_matvec(ctx, 1, x, prec)
            for q in range(3):
                want = vd.matvec_rows((eps - 1).ravel(), pos, g.h, K0, x[q].reshape(3, -1), rows)
                err = np.abs(y[q].reshape(3, -1)[:, rows] - want)
                assert np.max(err) <= bar * np.max(np.abs(want))
    finally:
        V.vie_destroy(ctx)


@pytest.mark.parametrize("prec,tol", [(0, 1e-11), (1, 1e-9)])
@pytest.mark.parametrize("n", GRIDS)
def test_solves_satisfy_the_oracle_system(V, n, prec, tol):
    rng, g, eps = _body(n)
    k = np.array([0.6, 0.0, 0.8])
    chans = [(k, [0, 1, 0]), (k, [0.8, 0.5j, -0.6]), (-k, [0, 1j, 0])]
    chi = (eps - 1).ravel()
    pos = vd.voxel_centres(g.n, g.h, g.origin)
    rows = rng.choice(np.nonzero(chi)[0], 40, replace=False)
    ctx = V.vie_setup([(eps, g.h, g.origin)],
                      V.make_options(K0, precision=prec, tol=tol, max_iter=4000))
    try:
        _, st = V.vie_solve(ctx, chans, [3])
        for q, (kh, p) in enumerate(chans):
            w = V.vie_get_current(ctx, 0, q, g.n).reshape(3, -1)
            b = vd.rhs(chi, pos, K0, kh, p)
            res = b[:, rows] - vd.matvec_rows(chi, pos, g.h, K0, w, rows)
            # sampled rows carry their share of the squared residual
            share = np.sqrt(len(rows) / np.count_nonzero(chi))
            assert np.linalg.norm(res) <= 2 * tol * np.linalg.norm(b) * max(5 * share, 1e-3)
    finally:
        V.vie_destroy(ctx)


@pytest.mark.parametrize("prec,tol", [(0, 1e-11), (1, 1e-9)])
@pytest.mark.parametrize("n", [g for g in GRIDS if g != (32, 32, 20)])
def test_solves_meet_their_tolerance_on_every_row(V, n, prec, tol):
    """The oracle's residual over all rows: at most the tolerance, and as much again for the
    rounding of both sides' operators."""
    rng, g, eps = _body(n)
    k = np.array([0.6, 0.0, 0.8])
    chi = (eps - 1).ravel()
    pos = vd.voxel_centres(g.n, g.h, g.origin)
    ctx = V.vie_setup([(eps, g.h, g.origin)],
                      V.make_options(K0, precision=prec, tol=tol, max_iter=4000))
    try:
        V.vie_solve(ctx, [(k, [0.8, 0.5j, -0.6])], [1])
        w = V.vie_get_current(ctx, 0, 0, g.n).reshape(3, -1)
    finally:
        V.vie_destroy(ctx)
    b = vd.rhs(chi, pos, K0, k, [0.8, 0.5j, -0.6])
    res = np.linalg.norm(b - vd.matvec(chi, pos, g.h, K0, w)) / np.linalg.norm(b)
    print(n, prec, res)
    assert res <= 2 * tol
