"""GPU parity of the block-Jacobi preconditioner and restarted flexible GMRES
(the block preconditioner of the large metasurface solve, Sec. III-B; FGMRES
after Saad 1993) against the oracle (dense block systems, k-step GMRES
block solves, textbook FGMRES).

* vie_precond_apply equals the oracle's block Jacobi with k-step GMRES block
  solves (FP64 products: rel. 1e-9; FP32 block products: rel. 1e-5; FP32
  products with the block basis stored in bfloat16: rel. 2e-2, a few
  bfloat16 unit roundoffs 2^-9 amplified by the small-k GMRES), and with k
  at least the block dimension, the exact block inverse;
* a fixed number of FGMRES steps (one cycle, and several restarted cycles)
  gives the oracle's iterate (both are the same function of the data in
  exact arithmetic; rel. 1e-8);
* converged solves equal the dense LU solution (FP64 to 1e-10: rel. 1e-8;
  mixed to 1e-6: rel. 1e-5, also with the bfloat16 block basis), with and
  without the preconditioner;
* several bodies on several grids in one call; the learned warm start with
  its fallback;
* the packed-FP16 z pass of the block products (VIE_MIXED_BF16 on a block
  grid that takes it, FFT 128 x 128 x 64): the preconditioner agrees with the
  FP32 block products to 2e-2 (FP16 unit roundoff 2^-11 through six pruned
  64-point transforms, plus the bfloat16 basis), and a converged solve
  satisfies the oracle's system on sampled rows (residual 2e-6 at tol 1e-6);
* option checks.
"""

import numpy as np
import pytest
import scipy.linalg

from oracle import precond as pc
from oracle import vie_dense as vd
from synth import Grid, random_ellipsoid_body

pytestmark = pytest.mark.gpu
K0 = 2 * np.pi
CHANS = [((0.0, 0.6, 0.8), (1.0, 0.0, 0.0)), ((0.0, 0.0, 1.0), (0.3, 1j, 0.0))]


@pytest.fixture(scope="module")
def V():
    import torch

    assert torch.cuda.is_available()
    from paper_2508_16471_amd import vie

    vie.lib()
    return vie


def _case(seed, n=(14, 11, 5), h=0.07):
    rng = np.random.default_rng(seed)
    g = Grid.centred(n, h)
    eps = random_ellipsoid_body(rng, g, kmax=3, axis_range=(0.25, 0.6))
    chi = (eps - 1.0).ravel()
    pos = vd.voxel_centres(g.n, g.h, g.origin)
    A, body = vd.body_system(chi, pos, g.h, K0)
    return g, eps, chi, pos, A, body


def _ctx(V, g, eps, precision, tol=1e-10, max_iter=2000):
    opt = V.make_options(K0, precision=precision, tol=tol, max_iter=max_iter)
    return V.vie_setup([(eps, g.h, g.origin)], opt)


def _body_vec(w, body):
    return w.reshape(3, -1)[:, body].reshape(-1)


def _rhs(chi, pos, body, k, p):
    return vd.rhs(chi, pos, K0, k, p)[:, body].reshape(-1)


@pytest.mark.parametrize("blocks,k,prec,tol", [((3, 2), 3, 0, 1e-9), ((7, 7), 2, 0, 1e-9),
                                               ((2, 3), 4, 1, 1e-5), ((1, 1), 5, 0, 1e-9),
                                               ((2, 3), 4, 2, 2e-2), ((7, 7), 3, 2, 2e-2)])
def test_precond_apply_matches_oracle(V, blocks, k, prec, tol):
    g, eps, chi, pos, A, body = _case(11)
    rng = np.random.default_rng(5)
    r = rng.standard_normal((2, 3) + g.n[::-1]) + 1j * rng.standard_normal((2, 3) + g.n[::-1])
    bset = pc.block_index_sets(pc.lateral_blocks(g.n, *blocks)[body])
    ctx = _ctx(V, g, eps, V.VIE_FP64)
    try:
        z = V.vie_precond_apply(ctx, V.fgmres_options(blocks=blocks, inner_iters=k,
                                                      inner_precision=prec), r)
    finally:
        V.vie_destroy(ctx)
    off = np.ones(int(np.prod(g.n)), bool)
    off[body] = False
    for q in range(2):
        want = pc.block_jacobi(A, bset, _body_vec(r[q], body), k=k)
        got = _body_vec(z[q], body)
        err = np.linalg.norm(got - want) / np.linalg.norm(want)
        print(blocks, k, prec, q, err)
        assert err < tol
        assert np.all(z[q].reshape(3, -1)[:, off] == 0)


def test_precond_exact_block_inverse(V):
    """k >= the largest block's unknown count: k-step GMRES is exact."""
    g, eps, chi, pos, A, body = _case(12, n=(14, 14, 3))
    bset = pc.block_index_sets(pc.lateral_blocks(g.n, 7, 7)[body])
    assert max(len(i) for i in bset.values()) <= 64
    rng = np.random.default_rng(6)
    r = rng.standard_normal((3,) + g.n[::-1]) + 1j * rng.standard_normal((3,) + g.n[::-1])
    ctx = _ctx(V, g, eps, V.VIE_FP64)
    try:
        z = V.vie_precond_apply(ctx, V.fgmres_options(blocks=(7, 7), inner_iters=64,
                                                      inner_precision=V.VIE_FP64), r)
    finally:
        V.vie_destroy(ctx)
    want = pc.block_jacobi(A, bset, _body_vec(r, body))
    err = np.linalg.norm(_body_vec(z, body) - want) / np.linalg.norm(want)
    print("exact block inverse", err)
    assert err < 1e-9


@pytest.mark.parametrize("restart,steps,blocks", [(8, 5, (3, 2)), (3, 7, (3, 2)), (4, 6, (0, 0))])
def test_fgmres_fixed_steps_match_oracle(V, restart, steps, blocks):
    g, eps, chi, pos, A, body = _case(13)
    k = 3
    ctx = _ctx(V, g, eps, V.VIE_FP64, tol=1e-15, max_iter=steps)
    fo = V.fgmres_options(restart=restart, blocks=blocks, inner_iters=k, inner_precision=V.VIE_FP64)
    try:
        rc, st = V.vie_solve_fgmres(ctx, CHANS, [2], fo, allow_noconv=True)
        ws = [_body_vec(V.vie_get_current(ctx, 0, q, g.n), body) for q in range(2)]
    finally:
        V.vie_destroy(ctx)
    M = None
    if blocks[0]:
        bset = pc.block_index_sets(pc.lateral_blocks(g.n, *blocks)[body])
        M = lambda v: pc.block_jacobi(A, bset, v, k=k)  # noqa: E731
    for q, (kh, p) in enumerate(CHANS):
        b = _rhs(chi, pos, body, kh, p)
        x, it, hist = pc.fgmres(lambda v: A @ v, b, M, m=restart, tol=1e-15, maxit=steps)
        err = np.linalg.norm(ws[q] - x) / np.linalg.norm(x)
        res = np.linalg.norm(b - A @ ws[q]) / np.linalg.norm(b)
        print(restart, steps, blocks, q, st[q]["iters"], it, err, res, st[q]["rel_res"], hist[-1])
        assert st[q]["iters"] == it == steps
        assert err < 1e-8
        assert abs(st[q]["rel_res"] - res) < 1e-9 * max(res, 1e-3)


@pytest.mark.parametrize("prec,inner,tol,blocks", [(0, 0, 1e-10, (3, 2)), (1, 1, 1e-6, (3, 2)),
                                                   (0, 0, 1e-10, (0, 0)), (1, 1, 1e-6, (7, 7)),
                                                   (1, 2, 1e-6, (3, 2)), (0, 2, 1e-10, (2, 2))])
def test_fgmres_converges_to_lu(V, prec, inner, tol, blocks):
    g, eps, chi, pos, A, body = _case(14)
    ctx = _ctx(V, g, eps, prec, tol=tol)
    fo = V.fgmres_options(restart=10, blocks=blocks, inner_iters=3, inner_precision=inner)
    try:
        rc, st = V.vie_solve_fgmres(ctx, CHANS, [2], fo)
        ws = [V.vie_get_current(ctx, 0, q, g.n) for q in range(2)]
    finally:
        V.vie_destroy(ctx)
    lu = scipy.linalg.lu_factor(A)
    for q, (kh, p) in enumerate(CHANS):
        b = _rhs(chi, pos, body, kh, p)
        want = scipy.linalg.lu_solve(lu, b)
        got = _body_vec(ws[q], body)
        err = np.linalg.norm(got - want) / np.linalg.norm(want)
        res = np.linalg.norm(b - A @ got) / np.linalg.norm(b)
        print(prec, inner, blocks, q, st[q], err, res)
        assert rc == 0 and st[q]["converged"] and st[q]["rel_res"] <= tol
        assert res <= tol * 1.01
        assert err < (1e-8 if prec == 0 else 1e-5)


def test_fgmres_rejects_bad_options(V):
    g, eps, chi, pos, A, body = _case(15, n=(6, 5, 4))
    ctx = _ctx(V, g, eps, V.VIE_FP64)
    try:
        for kw in [dict(restart=0), dict(restart=129), dict(blocks=(7, 2)), dict(blocks=(0, 2)),
                   dict(blocks=(2, 2), inner_iters=0), dict(blocks=(2, 2), inner_iters=65),
                   dict(blocks=(2, 2), inner_precision=3)]:
            with pytest.raises(V.VieError) as e:
                V.vie_solve_fgmres(ctx, CHANS[:1], [1], V.fgmres_options(**kw))
            assert e.value.code == V.VIE_EINVAL, kw
        with pytest.raises(V.VieError) as e:
            V.vie_precond_apply(ctx, V.fgmres_options(blocks=(0, 0)),
                                np.zeros((3,) + g.n[::-1], complex))
        assert e.value.code == V.VIE_EINVAL
    finally:
        V.vie_destroy(ctx)
    ctx = V.vie_setup([(eps, g.h, g.origin), (eps, g.h, g.origin)],
                      V.make_options(K0, tol=1e-6, max_iter=100))
    try:
        with pytest.raises(V.VieError) as e:  # the preconditioner alone takes one body
            V.vie_precond_apply(ctx, V.fgmres_options(blocks=(2, 2)),
                                np.zeros((3,) + g.n[::-1], complex))
        assert e.value.code == V.VIE_ENOTSUP
    finally:
        V.vie_destroy(ctx)


@pytest.mark.parametrize("prec,tol", [(0, 1e-10), (1, 1e-6)])
def test_fgmres_several_bodies_and_grids(V, prec, tol):
    """Three bodies in two grid groups (two share a grid), uneven channel
    counts: one batched FGMRES call with the block preconditioner; every
    solution equals its body's LU solution."""
    cases = [_case(21), _case(22), _case(23, n=(9, 12, 6))]
    bodies = [(c[1], c[0].h, c[0].origin) for c in cases]
    nrhs = [2, 1, 2]
    chans = CHANS[:2] + CHANS[:1] + CHANS[:2]
    opt = V.make_options(K0, precision=prec, tol=tol, max_iter=2000)
    ctx = V.vie_setup(bodies, opt)
    try:
        rc, st = V.vie_solve_fgmres(ctx, chans, nrhs,
                                    V.fgmres_options(6, (2, 2), 3, inner_precision=prec))
        assert rc == 0 and all(s["converged"] and s["rel_res"] <= tol for s in st)
        i = 0
        for b, (g, eps, chi, pos, A, body) in enumerate(cases):
            lu = scipy.linalg.lu_factor(A)
            for q in range(nrhs[b]):
                kh, p = chans[i]
                want = scipy.linalg.lu_solve(lu, _rhs(chi, pos, body, kh, p))
                got = _body_vec(V.vie_get_current(ctx, b, q, g.n), body)
                err = np.linalg.norm(got - want) / np.linalg.norm(want)
                print(b, q, st[i]["iters"], err)
                assert err < (1e-8 if prec == 0 else 1e-5)
                i += 1
    finally:
        V.vie_destroy(ctx)


def test_fgmres_warm_start_fallback(V):
    """An untrained network's guesses are checked like the BiCGSTAB path's: a
    guess with ||b - A x0|| >= ||b|| falls back to w = 0; the solve still
    meets the tolerance."""
    g, eps, chi, pos, A, body = _case(24)
    net = V.vie_cnn_create(3)
    opt = V.make_options(K0, precision=V.VIE_MIXED, tol=1e-6, max_iter=2000, warm_start=1)
    ctx = V.vie_setup([(eps, g.h, g.origin)], opt)
    try:
        V.vie_attach_cnn(ctx, net)
        rc, st = V.vie_solve_fgmres(ctx, CHANS, [2], V.fgmres_options(8, (2, 2), 3))
        print(st)
        assert rc == 0 and all(s["converged"] and s["warm"] == 1 for s in st)
        for s in st:
            assert s["fallback"] == (1 if s["rel_res_x0"] >= 1.0 else 0)
    finally:
        V.vie_destroy(ctx)
        V.vie_cnn_destroy(net)


def test_fgmres_empty_body_and_silent_body(V):
    """A body without voxels (eps = 1 everywhere) converges at once with w = 0;
    a body given no channels is skipped; the third body still matches LU."""
    g, eps, chi, pos, A, body = _case(25)
    empty = np.ones_like(eps)
    bodies = [(empty, g.h, g.origin), (eps, g.h, g.origin), (eps, g.h, g.origin)]
    ctx = V.vie_setup(bodies, V.make_options(K0, precision=V.VIE_FP64, tol=1e-10, max_iter=2000))
    try:
        rc, st = V.vie_solve_fgmres(ctx, CHANS[:2], [1, 0, 1], V.fgmres_options(8, (2, 2), 3))
        assert rc == 0 and st[0]["converged"] and st[0]["iters"] == 0 and st[0]["rel_res"] == 0
        w0 = V.vie_get_current(ctx, 0, 0, g.n)
        assert np.all(w0 == 0)
        kh, p = CHANS[1]
        want = scipy.linalg.lu_solve(scipy.linalg.lu_factor(A), _rhs(chi, pos, body, kh, p))
        got = _body_vec(V.vie_get_current(ctx, 2, 0, g.n), body)
        assert np.linalg.norm(got - want) < 1e-8 * np.linalg.norm(want)
    finally:
        V.vie_destroy(ctx)


# block boxes 60 x 60 x 29 (FFT 128 x 128 x 64: fused x-y passes) and
# 32 x 24 x 40 (FFT 64 x 48 x 96: 3 * 2^k lines in y and z, separate passes)
@pytest.mark.parametrize("n,fused", [((120, 120, 29), True), ((64, 48, 40), False)])
def test_packed_fp16_block_products(V, n, fused):
    rng = np.random.default_rng(41)
    h = 0.03
    g = Grid.centred(n, h)
    eps = 1.0 + rng.uniform(0.5, 2.0, size=n[::-1])
    eps[rng.random(eps.shape) < 0.2] = 1.0
    chi = (eps - 1.0).ravel()
    r = rng.standard_normal((1, 3) + n[::-1]) + 1j * rng.standard_normal((1, 3) + n[::-1])
    out = {}
    for inner in (V.VIE_MIXED, V.VIE_MIXED_BF16):
        ctx = V.vie_setup([(eps, h, g.origin)],
                          V.make_options(K0, precision=V.VIE_MIXED, flags=V.VIE_FLAG_TIMING))
        try:
            fo = V.fgmres_options(blocks=(2, 2), inner_iters=8, inner_precision=inner)
            out[inner] = V.vie_precond_apply(ctx, fo, r)
            t = V.vie_kernel_times(ctx, reset=True)
        finally:
            V.vie_destroy(ctx)
        passes = ("x_fwd", "y_fwd", "z", "y_inv", "x_inv")
        n16 = {k: t["block_fft_%s_h16" % k][1] for k in passes + ("xy_fwd", "yx_inv")}
        n32 = [t["block_fft_%s_f32" % ("z_green" if k == "z" else k)][1] for k in passes]
        print(inner, "block launches fp32", n32, "packed fp16", n16)
        packed = inner == V.VIE_MIXED_BF16
        want = ({"xy_fwd", "z", "yx_inv"} if fused else set(passes)) if packed else set()
        assert {k for k, c in n16.items() if c > 0} == want
        assert all((c > 0) != packed for c in n32)
    e = np.linalg.norm(out[V.VIE_MIXED_BF16] - out[V.VIE_MIXED]) / np.linalg.norm(out[V.VIE_MIXED])
    print("packed-FP16 preconditioner vs FP32", e)
    assert e < 2e-2
    ctx = V.vie_setup([(eps, h, g.origin)], V.make_options(K0, precision=V.VIE_MIXED, tol=1e-6,
                                                          max_iter=5000))
    try:
        rc, st = V.vie_solve_fgmres(ctx, CHANS[:1], [1],
                                    V.fgmres_options(30, (2, 2), 8, V.VIE_MIXED_BF16))
        w = V.vie_get_current(ctx, 0, 0, g.n).reshape(3, -1)
    finally:
        V.vie_destroy(ctx)
    print("solve", st[0])
    assert rc == 0 and st[0]["converged"] and st[0]["rel_res"] <= 1e-6
    pos = vd.voxel_centres(g.n, g.h, g.origin)
    body = np.nonzero(chi)[0]
    rows = np.unique(np.concatenate([rng.choice(body, 24, replace=False), body[[0, -1]]]))
    kh, p = CHANS[0]
    aw = vd.matvec_rows(chi, pos, h, K0, w, rows)
    b = vd.rhs(chi, pos, K0, kh, p)[:, rows]
    res = float(np.linalg.norm(b - aw) / np.linalg.norm(b))
    print("sampled residual", res)
    assert res < 2e-6


# block boxes at the edges of the fused x-y lengths (64: 25..32 cells, 96: 33..48, 128: 49..64),
# uneven in x and y, with z lines that are full (16, 32, 48 cells) or padded (29, 33, 40)
@pytest.mark.parametrize("n", [(50, 50, 29), (64, 50, 32), (63, 96, 40), (66, 128, 33),
                               (96, 50, 48), (97, 70, 16), (128, 98, 32), (128, 128, 29)])
def test_packed_fp16_planes_of_every_length(V, n):
    """Two block GMRES steps against FP64 ones.  The basis is rounded to bfloat16 (2^-9 a
    vector, two vectors, once more through the product of the first), the FP16 transforms add
    a few 2^-11: below 1e-2 in all."""
    print("packed planes", n, flush=True)
    rng = np.random.default_rng(7)
    h = 0.03
    g = Grid.centred(n, h)
    eps = 1.0 + rng.uniform(0.5, 2.0, size=n[::-1])
    eps[rng.random(eps.shape) < 0.3] = 1.0
    r = rng.standard_normal((2, 3) + n[::-1]) + 1j * rng.standard_normal((2, 3) + n[::-1])
    out = {}
    for prec, inner in ((V.VIE_FP64, V.VIE_FP64), (V.VIE_MIXED, V.VIE_MIXED_BF16)):
        ctx = V.vie_setup([(eps, h, g.origin)],
                          V.make_options(K0, precision=prec, flags=V.VIE_FLAG_TIMING))
        try:
            out[inner] = V.vie_precond_apply(
                ctx, V.fgmres_options(blocks=(2, 2), inner_iters=2, inner_precision=inner), r)
            t = V.vie_kernel_times(ctx, reset=True)
        finally:
            V.vie_destroy(ctx)
        assert (t["block_fft_xy_fwd_h16"][1] > 0) == (inner == V.VIE_MIXED_BF16)
    for q in range(2):
        e = (np.linalg.norm(out[V.VIE_MIXED_BF16][q] - out[V.VIE_FP64][q])
             / np.linalg.norm(out[V.VIE_FP64][q]))
        print("error", q, e)
        assert e < 1e-2


@pytest.mark.parametrize("k", [1, 31, 32, 33])
def test_block_least_squares_of_every_size(V, k):
    """Block solves whose least squares fit one wave's LDS (k <= 32) and one that does not,
    against the oracle's k-step GMRES (bar as the other FP64 block solves)."""
    print("block steps", k, flush=True)
    g, eps, chi, pos, A, body = _case(11)
    rng = np.random.default_rng(8)
    r = rng.standard_normal((2, 3) + g.n[::-1]) + 1j * rng.standard_normal((2, 3) + g.n[::-1])
    bset = pc.block_index_sets(pc.lateral_blocks(g.n, 3, 2)[body])
    ctx = _ctx(V, g, eps, V.VIE_FP64)
    try:
        z = V.vie_precond_apply(ctx, V.fgmres_options(blocks=(3, 2), inner_iters=k,
                                                      inner_precision=V.VIE_FP64), r)
    finally:
        V.vie_destroy(ctx)
    for q in range(2):
        want = pc.block_jacobi(A, bset, _body_vec(r[q], body), k=k)
        err = np.linalg.norm(_body_vec(z[q], body) - want) / np.linalg.norm(want)
        print(q, err)
        assert err < 1e-9


def test_steps_of_few_and_many_right_hand_sides(V):
    """16 right-hand sides take a wave each, 17 a lane each: the same iterates after six steps
    (FP64 roundings of the products, at most 1e-14 a step, through six steps)."""
    g, eps, chi, pos, A, body = _case(13)
    rng = np.random.default_rng(9)
    chans = []
    for _ in range(17):
        k = rng.standard_normal(3)
        k /= np.linalg.norm(k)
        p = np.cross(k, rng.standard_normal(3)) + 0j
        chans.append((k, p / np.linalg.norm(p)))
    w = {}
    for n in (1, 16, 17):
        ctx = _ctx(V, g, eps, V.VIE_FP64, tol=1e-15, max_iter=6)
        try:
            V.vie_solve_fgmres(ctx, chans[:n], [n], V.fgmres_options(4, (0, 0), 1, V.VIE_FP64),
                               allow_noconv=True)
            w[n] = [V.vie_get_current(ctx, 0, q, g.n) for q in range(n)]
        finally:
            V.vie_destroy(ctx)
    for q in range(16):
        assert np.linalg.norm(w[16][q] - w[17][q]) <= 1e-11 * np.linalg.norm(w[17][q])
    assert np.linalg.norm(w[1][0] - w[17][0]) <= 1e-11 * np.linalg.norm(w[17][0])


# block boxes of every y and z FFT length (y: 25..32, 33..48, 49..64 cells; z: 16, 25..32,
# 33..48, 49..64) and uneven x, lines full or padded
@pytest.mark.parametrize("n", [(104, 52, 16), (108, 112, 16), (52, 70, 30), (56, 60, 64),
                               (100, 80, 53), (54, 128, 64), (70, 99, 49), (104, 64, 41),
                               (90, 67, 46), (128, 105, 34)])
def test_packed_fp16_lines_of_every_length(V, n):
    """Every line along x, y and z of a two-step block solve, against FP64 products.  An entry
    carries the rounding of two bfloat16 vectors (2^-9 each) and a few 2^-11 of the FP16
    transforms, of the size of its neighbours: 1e-2 of a line's own norm leaves a factor of two
    for entries that cancel.  A line left out, doubled, or at the wrong frequency is off by 0.1
    and more, which the norm of the whole vector would hide."""
    print("packed lines", n, flush=True)
    rng = np.random.default_rng(sum(n))
    h = 0.03
    g = Grid.centred(n, h)
    eps = 1.0 + rng.uniform(0.5, 2.0, size=n[::-1])
    eps[rng.random(eps.shape) < 0.3] = 1.0
    r = rng.standard_normal((1, 3) + n[::-1]) + 1j * rng.standard_normal((1, 3) + n[::-1])
    out = []
    for inner in (V.VIE_FP64, V.VIE_MIXED_BF16):
        ctx = V.vie_setup([(eps, h, g.origin)],
                          V.make_options(K0, precision=V.VIE_MIXED, flags=V.VIE_FLAG_TIMING))
        try:
            out.append(V.vie_precond_apply(
                ctx, V.fgmres_options(blocks=(2, 2), inner_iters=2, inner_precision=inner), r)[0])
            t = V.vie_kernel_times(ctx, reset=True)
        finally:
            V.vie_destroy(ctx)
        assert (t["block_fft_xy_fwd_h16"][1] > 0) == (inner == V.VIE_MIXED_BF16)
    body = eps != 1.0
    for ax in (1, 2, 3):
        e = np.sqrt((np.abs(out[1] - out[0]) ** 2).sum(ax) / np.maximum(
            (np.abs(out[0]) ** 2).sum(ax), 1e-300))
        full = np.broadcast_to(body.sum(ax - 1) >= 6, e.shape)
        print("axis", "zyx"[ax - 1], "largest error of a line", e[full].max())
        assert full.any() and e[full].max() < 1e-2
