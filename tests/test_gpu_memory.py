"""Calls that do not fit the device's memory are refused with VIE_ENOMEM and leave
the handle usable: the next call of ordinary size gives what it gave before.
Nothing is launched by a refused call.  Where a call's own size does not exceed
the card, the rest of the card's memory is taken first (`short_of_memory`)."""

import contextlib

import numpy as np
import pytest

from synth import Grid, sphere

pytestmark = pytest.mark.gpu
K0 = 2 * np.pi
MIB = 1 << 20


@pytest.fixture(scope="module")
def V():
    import torch

    assert torch.cuda.is_available()
    from paper_2508_16471_amd import vie

    vie.lib()
    return vie


@contextlib.contextmanager
def short_of_memory(left):
    """Takes all device memory but about `left` bytes."""
    import torch

    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    try:
        for piece in (8192 * MIB, 1024 * MIB, 128 * MIB, 32 * MIB):
            while torch.cuda.mem_get_info()[0] > left + piece:
                held.append(torch.empty(piece, dtype=torch.uint8, device="cuda"))
        yield
    finally:
        held.clear()
        torch.cuda.empty_cache()


def _channels(n):
    rng = np.random.default_rng(n)
    out = []
    for _ in range(n):
        k = rng.standard_normal(3)
        k /= np.linalg.norm(k)
        p = np.cross(k, rng.standard_normal(3))
        out.append((k, p / np.linalg.norm(p)))
    return out


def test_product_after_one_that_does_not_fit(V):
    """20000 vectors of 128 x 128 x 16 want 500 GB for their x lines alone."""
    import torch

    g = Grid.centred((128, 128, 16), 1 / 32)
    rng = np.random.default_rng(3)
    eps = np.where(rng.random(g.n[::-1]) < 0.5, 2.0, 1.0)
    x = torch.randn((2, 3) + eps.shape, dtype=torch.complex128, device="cuda")
    y, z = torch.empty_like(x), torch.empty_like(x)
    ctx = V.vie_setup([(eps, g.h, g.origin)], V.make_options(K0))
    try:
        print("product of two vectors, then of too many", flush=True)
        V.vie_matvec_dev(ctx, 0, x.data_ptr(), y.data_ptr(), 2)
        assert V.lib().vie_matvec_dev(ctx, 0, V.VIE_FP64, x.data_ptr(), z.data_ptr(),
                                      20000) == V.VIE_ENOMEM
        V.vie_matvec_dev(ctx, 0, x.data_ptr(), z.data_ptr(), 2)
        torch.cuda.synchronize()
        assert torch.equal(y, z)
    finally:
        V.vie_destroy(ctx)


def test_solve_after_one_that_does_not_fit(V):
    """A refused solve leaves no solution behind (VIE_ESTATE, not a read of
    released memory) and the next one finds its own."""
    g = Grid.centred(48, 1 / 16)
    eps = sphere(g, 1.2, 2.25)
    th = np.linspace(0.1, 3.0, 7)
    ctx = V.vie_setup([(eps, g.h, g.origin)], V.make_options(K0, tol=1e-8, max_iter=2000))
    try:
        print("solve of one channel, then of many without memory", flush=True)
        V.vie_solve(ctx, _channels(1), [1])
        F = V.vie_farfield(ctx, 0, th, th, 1)
        with short_of_memory(512 * MIB):
            with pytest.raises(V.VieError) as e:
                V.vie_solve(ctx, _channels(64), [64])
            assert e.value.code == V.VIE_ENOMEM
            with pytest.raises(V.VieError) as e:
                V.vie_farfield(ctx, 0, th, th, 1)
            assert e.value.code in (V.VIE_EINVAL, V.VIE_ESTATE)
        V.vie_solve(ctx, _channels(1), [1])
        assert np.array_equal(V.vie_farfield(ctx, 0, th, th, 1), F)
    finally:
        V.vie_destroy(ctx)


def test_rooftop_setup_after_one_that_does_not_fit(V):
    """Setting up 128^3 wants gigabytes; refused, it leaves the runtime clean
    for the calls of another operator."""
    g = Grid.centred((12, 9, 10), 0.05)
    eps = np.full(g.n[::-1], 2.0)
    x = np.random.default_rng(1).standard_normal((1, 3, 12, 11, 14)) + 0j
    r = V.vie_rt_setup(eps, g.h, g.origin, K0)
    try:
        print("rooftop product beside a setup without memory", flush=True)
        y = V.vie_rt_matvec(r, x)
        with short_of_memory(512 * MIB):
            with pytest.raises(V.VieError) as e:
                V.vie_rt_setup(np.full((128, 128, 128), 2.0), 0.05, (0, 0, 0), K0)
            assert e.value.code == V.VIE_ENOMEM
            assert np.array_equal(V.vie_rt_matvec(r, x), y)
    finally:
        V.vie_rt_destroy(r)


def test_network_after_a_box_that_does_not_fit(V):
    import torch

    net = V.vie_cnn_create(1)
    feat = torch.randn((16, 512, 512, 32), dtype=torch.bfloat16, device="cuda")
    out, again = (torch.empty((16, 512, 512, 16), device="cuda") for _ in range(2))
    small, big = (9, 8, 7), (512, 512, 16)
    n = 9 * 8 * 7 * 16
    try:
        print("network, then a box without memory", flush=True)
        V.vie_cnn_infer_dev(net, small, feat.data_ptr(), out.data_ptr())
        with short_of_memory(512 * MIB):  # its layers want 1.6 GB
            with pytest.raises(V.VieError) as e:
                V.vie_cnn_infer_dev(net, big, feat.data_ptr(), again.data_ptr())
            assert e.value.code == V.VIE_ENOMEM
        V.vie_cnn_infer_dev(net, small, feat.data_ptr(), again.data_ptr())
        torch.cuda.synchronize()
        assert torch.equal(out.ravel()[:n], again.ravel()[:n])
    finally:
        V.vie_cnn_destroy(net)


def test_sample_after_products_of_more_vectors(V, monkeypatch):
    """Products between a solve and its training sample, with more vectors than
    the solve had channels: the sample is that of the solve, bit for bit."""
    import torch

    monkeypatch.setenv("VIE_DETERMINISTIC", "1")

    g = Grid.centred(20, 1 / 16)
    eps = sphere(g, 0.55, 2.25)
    x = torch.randn((40, 3) + eps.shape, dtype=torch.complex128, device="cuda")
    y = torch.empty_like(x)
    got = []
    for products in (0, 1, 40):
        print("sample after a product of", products, flush=True)
        ctx = V.vie_setup([(eps, g.h, g.origin)], V.make_options(K0, tol=1e-8, max_iter=2000))
        try:
            V.vie_solve(ctx, _channels(2), [2])
            if products:
                V.vie_matvec_dev(ctx, 0, x.data_ptr(), y.data_ptr(), products)
            d = V.vie_cnn_sample_dev(ctx, 0, 1)
            feat = torch.zeros(d[::-1] + (32,), dtype=torch.bfloat16, device="cuda")
            target = torch.zeros(d[::-1] + (6,), device="cuda")
            V.vie_cnn_sample_dev(ctx, 0, 1, feat.data_ptr(), target.data_ptr())
            torch.cuda.synchronize()
            got.append((feat, target))
        finally:
            V.vie_destroy(ctx)
    assert got[0][1].abs().max() > 0
    for feat, target in got[1:]:
        assert torch.equal(feat, got[0][0]) and torch.equal(target, got[0][1])


def test_rooftop_calls_need_no_memory_beyond_setup(V):
    """A rooftop operator that could be set up multiplies and solves, whatever
    memory is left: 40 channels of 21 MB each run in smaller batches, to the
    same iterates."""
    g = Grid.centred((30, 28, 26), 1 / 16)
    eps = sphere(g, 0.7, 2.25)
    rng = np.random.default_rng(2)
    x = rng.standard_normal((2, 3, 28, 30, 32)) + 0j
    chans = _channels(40)
    r = V.vie_rt_setup(eps, g.h, g.origin, K0)
    try:
        print("rooftop calls with memory", flush=True)
        y = V.vie_rt_matvec(r, x)
        _, w, st = V.vie_rt_solve(r, chans, tol=1e-8, max_iter=500)
    finally:
        V.vie_rt_destroy(r)
    r = V.vie_rt_setup(eps, g.h, g.origin, K0)
    try:
        with short_of_memory(128 * MIB):
            print("rooftop calls without memory", flush=True)
            assert np.array_equal(V.vie_rt_matvec(r, x), y)
            _, w2, st2 = V.vie_rt_solve(r, chans, tol=1e-8, max_iter=500)
        assert np.array_equal(w2, w)
        assert [s["iters"] for s in st2] == [s["iters"] for s in st]
    finally:
        V.vie_rt_destroy(r)
