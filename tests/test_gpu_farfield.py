"""GPU parity of the far-field projection (eq. 25, FP64 MFMA contraction)
against the oracle's direct FP64 sum on the same currents w.

The currents come from the library's own solve (any iterate will do: the far
field is a linear map of w, and both sides read the same w).  Bodies are
chosen so that different voxel-block shapes win (x rod, y line, z column,
thin slab, blob), with ragged direction counts (1, 17, 181, 1000) and
right-hand-side counts (1, 3) that leave partial passes and partial tiles.
Bar: rel-L2 <= 1e-12 (FP64 everywhere; only the summation order differs).
"""

import numpy as np
import pytest

from oracle import vie_dense as vd
from synth import Grid, random_ellipsoid_body, sphere

pytestmark = pytest.mark.gpu
K0 = 2 * np.pi


@pytest.fixture(scope="module")
def V():
    import torch

    assert torch.cuda.is_available()
    from paper_2508_16471_amd import vie

    vie.lib()
    return vie


def _relerr(a, b):
    return float(np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b)))


def _body(kind, rng):
    if kind == "xrod":
        g = Grid.centred((37, 5, 4), 0.04)
        eps = np.ones((4, 5, 37))
        eps[2, 3, 1:36] = 3.0
    elif kind == "yline":
        g = Grid.centred((6, 41, 5), 0.04)
        eps = np.ones((5, 41, 6))
        eps[1, 2:39, 4] = 2.5
    elif kind == "zcol":
        g = Grid.centred((5, 4, 35), 0.04)
        eps = np.ones((35, 4, 5))
        eps[:, 1, 2] = 4.0
    elif kind == "slab":
        g = Grid.centred((21, 19, 3), 0.05)
        eps = np.ones((3, 19, 21))
        eps[1] = 2.1
    else:
        g = Grid.centred((18, 15, 13), 0.07)
        eps = random_ellipsoid_body(rng, g, kmax=3, axis_range=(0.2, 0.5))
    return g, eps


def _channels(rng, nrhs):
    out = []
    for _ in range(nrhs):
        k = rng.standard_normal(3)
        k /= np.linalg.norm(k)
        p = np.cross(k, rng.standard_normal(3))
        p /= np.linalg.norm(p)
        out.append((k, p + 0.3j * np.cross(k, p)))
    return out


@pytest.mark.parametrize("kind,nrhs,ndir", [("xrod", 1, 17), ("yline", 3, 1), ("zcol", 2, 181),
                                            ("slab", 3, 1000), ("blob", 2, 181)])
def test_farfield_matches_direct_sum(V, kind, nrhs, ndir):
    rng = np.random.default_rng(len(kind) * 100 + ndir)
    g, eps = _body(kind, rng)
    chans = _channels(rng, nrhs)
    theta = rng.uniform(0, np.pi, ndir)
    phi = rng.uniform(-np.pi, np.pi, ndir)
    ctx = V.vie_setup([(eps, g.h, g.origin)], V.make_options(K0, tol=1e-3, max_iter=60))
    try:
        V.vie_solve(ctx, chans, [nrhs], allow_noconv=True)
        F = V.vie_farfield(ctx, 0, theta, phi, nrhs)
        pos = vd.voxel_centres(g.n, g.h, g.origin)
        for q in range(nrhs):
            w = V.vie_get_current(ctx, 0, q, g.n).reshape(3, -1)
            ft, fp = vd.farfield(w, pos, g.h, K0, theta, phi)
            err = _relerr(F[q], np.stack([ft, fp], -1))
            print(kind, q, ndir, "far-field rel err", err)
            assert err < 1e-12
    finally:
        V.vie_destroy(ctx)


def test_farfield_full_sweep_sphere_64(V):
    """Sphere radius 1 lambda, eps 4, 64^3 grid, two channels at +-30 deg:
    the 360 x 180 sweep (64,800 directions) checked on 300 sampled
    directions against the direct sum; reciprocity-free symmetry check: the
    sweep's phi = 0 row equals a separate call on those directions."""
    g = Grid.centred((64, 64, 64), 2.05 / 64)
    eps = sphere(g, 1.0, 4.0)
    a = np.deg2rad(30)
    chans = [((np.sin(a), 0, np.cos(a)), (np.cos(a), 0, -np.sin(a))),
             ((-np.sin(a), 0, np.cos(a)), (np.cos(a), 0, np.sin(a)))]
    th1 = (np.arange(180) + 0.5) * np.pi / 180
    ph1 = np.arange(360) * 2 * np.pi / 360 - np.pi
    TH, PH = np.meshgrid(th1, ph1, indexing="ij")
    ctx = V.vie_setup([(eps, g.h, g.origin)], V.make_options(K0, precision=V.VIE_MIXED, tol=1e-6,
                                                            max_iter=12000))
    try:
        _, st = V.vie_solve(ctx, chans, [2])
        assert all(s["converged"] for s in st)
        F = V.vie_farfield(ctx, 0, TH.ravel(), PH.ravel(), 2)
        rng = np.random.default_rng(64)
        idx = rng.choice(TH.size, 300, replace=False)
        pos = vd.voxel_centres(g.n, g.h, g.origin)
        for q in range(2):
            w = V.vie_get_current(ctx, 0, q, g.n).reshape(3, -1)
            ft, fp = vd.farfield(w, pos, g.h, K0, TH.ravel()[idx], PH.ravel()[idx])
            err = _relerr(F[q, idx], np.stack([ft, fp], -1))
            print("sweep sample rel err", q, err)
            assert err < 1e-12
        row = np.nonzero(np.isclose(PH.ravel(), 0.0))[0]
        F2 = V.vie_farfield(ctx, 0, TH.ravel()[row], PH.ravel()[row], 2)
        assert _relerr(F[:, row], F2) < 1e-13
    finally:
        V.vie_destroy(ctx)


@pytest.mark.parametrize("nrhs,ndir", [(3, 5), (5, 40)])
def test_farfield_right_hand_sides_in_several_launches(V, nrhs, ndir):
    """Bodies whose packed operand exceeds the per-launch share: the
    right-hand sides go out in launches of two with a remainder, the vector
    offsets still hold after a product with more vectors has grown the
    context's tables, and every one matches the direct sum (bar as above)."""
    import torch

    rng = np.random.default_rng(nrhs)
    g = Grid.centred((96, 96, 64), 1 / 64)
    eps = np.full((64, 96, 96), 1.05)
    theta, phi = rng.uniform(0, np.pi, ndir), rng.uniform(-np.pi, np.pi, ndir)
    ctx = V.vie_setup([(eps, g.h, g.origin)], V.make_options(K0, tol=1e-9, max_iter=2))
    try:
        V.vie_solve(ctx, _channels(rng, nrhs), [nrhs], allow_noconv=True)
        x = torch.zeros((nrhs + 1, 3) + eps.shape, dtype=torch.complex128, device="cuda")
        y = torch.empty_like(x)
        V.vie_matvec_dev(ctx, 0, x.data_ptr(), y.data_ptr(), nrhs + 1)
        F = V.vie_farfield(ctx, 0, theta, phi, nrhs)
        pos = vd.voxel_centres(g.n, g.h, g.origin)
        some = rng.choice(ndir, 4, replace=False)
        for q in range(nrhs):
            w = V.vie_get_current(ctx, 0, q, g.n).reshape(3, -1)
            ft, fp = vd.farfield(w, pos, g.h, K0, theta[some], phi[some])
            assert _relerr(F[q][some], np.stack([ft, fp], -1)) < 1e-12
    finally:
        V.vie_destroy(ctx)


@pytest.mark.parametrize("order", ["theta", "phi", "shuffled", "uneven"])
@pytest.mark.parametrize("shape,window", [((21, 19, 13), 0), ((5, 70, 30), 1), ((97, 66, 1), 0)])
def test_farfield_sweep_by_theta_matches_direct_path(V, order, shape, window):
    """Directions sharing theta take the column path: same values as the
    direct path (calls of few directions each) and as the oracle's sum, for
    any order of the directions, group sizes around the 16- and 64-direction
    tiles, flat and tall bodies with holes, with and without the z window
    (bar as above)."""
    rng = np.random.default_rng(shape[0])
    g = Grid.centred(shape, 0.03)
    eps = np.where(rng.random(shape[::-1]) < 0.7, 1.05, 1.0)
    if window:
        eps[:4] = eps[-7:] = 1.0
    counts = np.full(67, 100) if order != "uneven" else np.array([1, 15, 16, 17, 63, 64, 65, 129,
                                                                  2000, 3000, 1500])
    theta = np.repeat(rng.uniform(0, np.pi, len(counts)), counts)
    phi = np.concatenate([np.linspace(-np.pi, np.pi, n, endpoint=False) for n in counts])
    if order == "phi":
        at = np.argsort(phi, kind="stable")
    elif order == "theta":
        at = np.arange(theta.size)
    else:
        at = rng.permutation(theta.size)
    theta, phi = theta[at], phi[at]
    assert 1.25 * theta.size * (eps > 1).sum() > 3e7  # large enough for the column path
    nrhs = 3
    opt = V.make_options(K0, tol=1e-9, max_iter=2, flags=V.VIE_FLAG_Z_WINDOW if window else 0)
    ctx = V.vie_setup([(eps, g.h, g.origin)], opt)
    try:
        V.vie_solve(ctx, _channels(rng, nrhs), [nrhs], allow_noconv=True)
        F = V.vie_farfield(ctx, 0, theta, phi, nrhs)
        D = np.concatenate([V.vie_farfield(ctx, 0, theta[a:a + 500], phi[a:a + 500], nrhs)
                            for a in range(0, theta.size, 500)], axis=1)
        pos = vd.voxel_centres(g.n, g.h, g.origin)
        some = rng.choice(theta.size, 20, replace=False)
        for q in range(nrhs):
            assert _relerr(F[q], D[q]) < 1e-12
            w = V.vie_get_current(ctx, 0, q, g.n).reshape(3, -1)
            ft, fp = vd.farfield(w, pos, g.h, K0, theta[some], phi[some])
            assert _relerr(F[q][some], np.stack([ft, fp], -1)) < 1e-12
    finally:
        V.vie_destroy(ctx)


@pytest.mark.parametrize("ndir", [1, 64, 65, 333])
def test_farfield_block_shapes_share_a_launch(V, ndir):
    """A slab, y lines and z columns in separate bands of layers: block shapes of one launch
    with different tile counts, the last split of each shape shorter than the others."""
    print(f"farfield shapes ndir={ndir}", flush=True)
    rng = np.random.default_rng(19)
    g = Grid.centred((45, 43, 40), 0.03)
    eps = np.ones(g.n[::-1])
    eps[0:4, 3:41, 2:44] = 2.0
    eps[8:12, :, 5::7] = 2.5
    eps[20:40, 4::6, 3::5] = 3.0
    ctx = V.vie_setup([(eps, g.h, g.origin)], V.make_options(K0, tol=1e-2, max_iter=3))
    try:
        chans = _channels(rng, 2)
        V.vie_solve(ctx, chans, [2], allow_noconv=True)
        th = np.arccos(rng.uniform(-1, 1, ndir))
        ph = rng.uniform(-np.pi, np.pi, ndir)
        F = V.vie_farfield(ctx, 0, th, ph, 2)
        pos = vd.voxel_centres(g.n, g.h, g.origin)
        for q in range(2):
            w = V.vie_get_current(ctx, 0, q, g.n).reshape(3, -1)
            ft, fp = vd.farfield(w, pos, g.h, K0, th, ph)
            assert _relerr(F[q], np.stack([ft, fp], -1)) < 1e-12
    finally:
        V.vie_destroy(ctx)


def test_phases_are_taken_about_the_coordinate_origin(V):
    """One voxel at the coordinate origin in the middle of a box of 127 voxels of
    k0 h = 20: no phase at all, while the box's corner is at 1300 rad.  Bar: the
    roundings of the direction frames, the projection and the constants, 16 of
    2^-53; relative to the corner the rounding of one phase is 1e-13."""
    print("far field of one voxel", flush=True)
    rng = np.random.default_rng(4)
    n, h = (127, 63, 9), 3.25
    origin = tuple(-h * (m // 2) for m in n)
    eps = np.ones(n[::-1])
    eps[4, 31, 63] = 1.5
    theta, phi = np.arccos(rng.uniform(-1, 1, 40)), rng.uniform(-np.pi, np.pi, 40)
    ctx = V.vie_setup([(eps, h, origin)], V.make_options(K0, tol=1e-9, max_iter=2))
    try:
        V.vie_solve(ctx, _channels(rng, 1), [1], allow_noconv=True)
        F = V.vie_farfield(ctx, 0, theta, phi, 1)[0]
        w = V.vie_get_current(ctx, 0, 0, n)[:, 4, 31, 63].astype(np.clongdouble)
    finally:
        V.vie_destroy(ctx)
    t, p = theta.astype(np.longdouble), phi.astype(np.longdouble)
    C = np.longdouble(K0) ** 2 * np.longdouble(h) ** 3 / (16 * np.arctan(np.longdouble(1)))
    ref = C * np.stack([np.cos(t) * (np.cos(p) * w[0] + np.sin(p) * w[1]) - np.sin(t) * w[2],
                        np.cos(p) * w[1] - np.sin(p) * w[0]], -1)
    err = float(np.max(np.abs(F - ref)) / np.max(np.abs(ref)))
    print(err)
    assert err < 16 * 2.0 ** -53
