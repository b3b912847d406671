"""The workloads this library is timed on, each one pass through its public calls.

Kinds of work (`kind` of a case):

* product      y = A x on device vectors (`vie_matvec_dev`), the call of a user's own Krylov method;
* solve        channels of a few bodies to a tight residual, then the 181-point detector scan of every
               body (`vie_solve`, `vie_solve_fgmres`, `vie_farfield`);
* farfield     the far field of a solved body: a detector scan, or a sphere sweep on a (theta, phi) grid;
* rt_product, rt_solve, rt_farfield   the same three steps in the rooftop basis (host vectors);
* cnn_infer, cnn_train   the warm-start network on a body's box: a prediction, one training step.

Solves run to residuals near the ones the parity tests use, so that the far field is determined to many
digits whatever path the iteration takes.  Bodies, grids and channels are those of `bench.py` and the
tests (sphere, ellipsoid unions at h = 1/16, fin metasurfaces at h = 1/32).
"""

import math

import numpy as np
import torch

from paper_2508_16471_amd import vie as V
from synth import Grid, metasurface_family, random_ellipsoid_body, sphere

K0 = 2 * math.pi


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # one product on the 16^3 sphere grid: launches and latency
        {"name": "product_sphere16", "kind": "product", "nx": 16, "ny": 16, "nz": 16, "nvec": 1},
        # the benchmark's isolated products: 8 vectors on the full 128^3 grid
        {"name": "product_128x8", "kind": "product", "nx": 128, "ny": 128, "nz": 128, "nvec": 8},
        # a single small body, two channels, plain FP64: the interactive call
        {"name": "solve_sphere16", "kind": "solve", "solver": "fp64", "body": "sphere", "n": 16,
         "bodies": 1, "channels": 2, "tol": 1e-12},
        # uneven bodies in one mixed-precision batch (32^3 and 48^3 grids, 4 channels each)
        {"name": "solve_uneven", "kind": "solve", "solver": "mixed", "body": "ellipsoids", "n": 32,
         "bodies": 4, "channels": 4, "tol": 1e-11},
        # the benchmark step: 4 metasurface bodies x 2 channels, block-Jacobi FGMRES on the z window
        {"name": "solve_metasurface128", "kind": "solve", "solver": "fgmres", "body": "metasurface",
         "n": 128, "bodies": 4, "channels": 2, "tol": 1e-11},
        # the 181-point detector scan of one metasurface body, 2 channels
        {"name": "scan_metasurface128", "kind": "farfield", "body": "metasurface", "n": 128,
         "channels": 2, "ntheta": 181, "nphi": 1},
        # the 180 x 360 sphere sweep of the same body
        {"name": "sweep_metasurface128", "kind": "farfield", "body": "metasurface", "n": 128,
         "channels": 2, "ntheta": 180, "nphi": 360},
        # rooftop basis: one product of a host vector on the 64^3 sphere
        {"name": "rt_product_64", "kind": "rt_product", "nx": 64, "ny": 64, "nz": 64, "nvec": 1},
        # rooftop basis: two channels of a small body on a ragged grid
        {"name": "rt_solve_ragged", "kind": "rt_solve", "nx": 26, "ny": 21, "nz": 17, "channels": 2,
         "mixed": False, "tol": 1e-11},
        # rooftop basis: the 180 x 360 sweep of two channels on the 64^3 sphere
        {"name": "rt_sweep_64", "kind": "rt_farfield", "nx": 64, "ny": 64, "nz": 64, "channels": 2,
         "ntheta": 180, "nphi": 360},
        # network prediction on the box of a 128-cell metasurface body
        {"name": "cnn_infer_128", "kind": "cnn_infer", "d0": 128, "d1": 128, "d2": 37},
        # one training step on a box of odd extents
        {"name": "cnn_train_odd", "kind": "cnn_train", "d0": 121, "d1": 107, "d2": 37},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_directions(rng):
    if rng.random() < 0.25:
        return {"ntheta": _log_int(rng, 64, 4096), "nphi": 0}
    return {"ntheta": _log_int(rng, 9, 180), "nphi": _log_int(rng, 1, 360)}


def draw(rng):
    kind = rng.choice(["product", "product", "solve", "solve", "farfield", "farfield", "rt_product",
                       "rt_solve", "rt_farfield", "cnn_infer", "cnn_train"])
    if kind == "product":
        c = {"kind": kind, "nx": _log_int(rng, 12, 128), "ny": _log_int(rng, 12, 128),
             "nz": _log_int(rng, 12, 128), "nvec": rng.randint(1, 8)}
    elif kind == "solve":
        solver = rng.choice(["fp64", "mixed", "fgmres"])
        if solver == "fp64":
            c = {"kind": kind, "solver": solver, "body": rng.choice(["sphere", "ellipsoids"]),
                 "n": rng.randint(12, 32), "bodies": 1, "channels": rng.randint(1, 3), "tol": 1e-12}
        elif solver == "mixed":
            c = {"kind": kind, "solver": solver, "body": "ellipsoids", "n": rng.randint(20, 32),
                 "bodies": rng.randint(2, 4), "channels": rng.randint(1, 4), "tol": 1e-11}
        else:
            c = {"kind": kind, "solver": solver, "body": "metasurface",
                 "n": 8 * rng.randint(8, 16), "bodies": rng.randint(1, 3),
                 "channels": rng.randint(1, 2), "tol": 1e-11}
    elif kind == "farfield":
        c = {"kind": kind, "body": "metasurface", "n": 8 * rng.randint(6, 16),
             "channels": rng.randint(1, 2), **_draw_directions(rng)}
    elif kind == "rt_product":
        c = {"kind": kind, "nx": _log_int(rng, 10, 64), "ny": _log_int(rng, 10, 64),
             "nz": _log_int(rng, 10, 64), "nvec": rng.randint(1, 2)}
    elif kind == "rt_solve":
        c = {"kind": kind, "nx": rng.randint(10, 26), "ny": rng.randint(10, 26),
             "nz": rng.randint(10, 26), "channels": rng.randint(1, 2),
             "mixed": rng.random() < 0.5, "tol": 1e-11}
    elif kind == "rt_farfield":
        c = {"kind": kind, "nx": _log_int(rng, 10, 64), "ny": _log_int(rng, 10, 64),
             "nz": _log_int(rng, 10, 64), "channels": rng.randint(1, 2), **_draw_directions(rng)}
    else:
        c = {"kind": kind, "d0": _log_int(rng, 12, 128), "d1": _log_int(rng, 12, 128),
             "d2": _log_int(rng, 9, 37)}
    return c


# ------------------------------------------------------------- seeded inputs
def _channel(rng, cap_deg=None):
    """Plane-wave channel: direction in a cap about +z (or anywhere), random elliptical polarisation."""
    if cap_deg is None:
        k = rng.standard_normal(3)
    else:
        ct, ph = rng.uniform(math.cos(math.radians(cap_deg)), 1.0), rng.uniform(0, 2 * math.pi)
        st = math.sqrt(1 - ct * ct)
        k = np.array([st * math.cos(ph), st * math.sin(ph), ct])
    k = k / np.linalg.norm(k)
    p = rng.standard_normal(3) + 1j * rng.standard_normal(3)
    p = p - k * (k @ p)
    return k, p / np.linalg.norm(p)


def _bodies(case, rng):
    """[(eps, h, origin)] and the channels of every body."""
    bodies, chans = [], []
    for b in range(case.get("bodies", 1)):
        if case["body"] == "metasurface":
            grid, eps = metasurface_family(rng, case["n"])
        elif case["body"] == "sphere":
            grid = Grid.centred(case["n"], 1.0 / 16)
            eps = sphere(grid, 0.5 * case["n"] / 16 * rng.uniform(0.9, 1.0), rng.uniform(2.0, 2.5))
        else:  # every other body on a grid half again as large
            grid = Grid.centred(case["n"] * (3 if b % 2 else 2) // 2, 1.0 / 16)
            eps = random_ellipsoid_body(rng, grid, eps_range=(1.5, 3.0))
        bodies.append((eps, grid.h, grid.origin))
        chans += [_channel(rng, 20.0 if case["body"] == "metasurface" else None)
                  for _ in range(case["channels"])]
    return bodies, chans


def _rt_body(case, rng):
    """Ellipsoid of eps 2.1..4 filling the grid at h = 1/31 (the 64-cell sphere of r = 1)."""
    n = (case["nx"], case["ny"], case["nz"])
    g = Grid.centred(n, 2.05 / 64)
    x, y, z = g.mesh()
    r = [0.97 * n[a] * g.h / 2 for a in range(3)]
    eps = np.ones(x.shape)
    eps[(x / r[0]) ** 2 + (y / r[1]) ** 2 + (z / r[2]) ** 2 <= 1] = rng.uniform(2.1, 4.0)
    return eps, g.h, g.origin


def _rt_current(case, rng, eps, h, origin):
    """A plane-wave current of the internal wavenumber on the faces of the body's cells."""
    e = np.pad(eps - 1.0, 1)
    w = np.zeros((case["channels"], 3) + e.shape, complex)
    ax = [origin[a] + h * (np.arange(e.shape[2 - a]) - 1) for a in range(3)]
    for q in range(case["channels"]):
        k, p = _channel(rng)
        k = K0 * math.sqrt(eps.max()) * k
        ph = (np.exp(1j * k[2] * ax[2])[:, None, None] * np.exp(1j * k[1] * ax[1])[None, :, None]
              * np.exp(1j * k[0] * ax[0])[None, None, :])
        for i in range(3):
            w[q, i] = p[i] * ph * (_rt_faces(e)[0][i] > 0)
    return w


def _directions(case):
    """A scan (theta over 0..180 deg in the xz plane), the (theta, phi) grid of a sphere sweep, or
    (nphi = 0) ntheta directions spread over the sphere on a spiral."""
    nt, nph = case["ntheta"], case["nphi"]
    if nph == 0:
        i = np.arange(nt) + 0.5
        return np.arccos(1.0 - 2.0 * i / nt), math.pi * (3.0 - math.sqrt(5.0)) * i % (2 * math.pi)
    if nph == 1:
        return np.linspace(0.0, math.pi, nt), np.zeros(nt)
    th = (np.arange(nt) + 0.5) * math.pi / nt
    ph = np.arange(nph) * 2 * math.pi / nph
    t, p = np.meshgrid(th, ph, indexing="ij")
    return t.ravel(), p.ravel()


SCAN = {"ntheta": 181, "nphi": 1}


def _cnn_box(case, rng):
    """Network input, target and weights: unit-rms fields on 40 % of the box, He-scaled weights."""
    d = (case["d0"], case["d1"], case["d2"])
    g = torch.Generator(device="cuda").manual_seed(int(rng.integers(1 << 31)))
    shape = d[::-1]
    body = torch.rand(shape, generator=g, device="cuda") < 0.4
    feat = torch.zeros(shape + (32,), device="cuda")
    feat[..., :25] = torch.randn(shape + (25,), generator=g, device="cuda")
    feat[..., 0] = 0.3 + torch.rand(shape, generator=g, device="cuda")
    feat = (feat * body[..., None]).to(torch.bfloat16).contiguous()
    target = (torch.randn(shape + (6,), generator=g, device="cuda") * body[..., None]).contiguous()
    return d, feat, target, body


# 32 -> 32 -> 32 -> 32 -> 16 channels, 27 taps: (W[27][Cout][Cin], b[Cout]) per layer
CNN_SHAPES = [((27, 32, 32), (32,))] * 3 + [((27, 16, 32), (16,))]


def _cnn_weights(rng):
    p = []
    for ws, bs in CNN_SHAPES:
        p += [rng.standard_normal(ws).ravel() * math.sqrt(2.0 / (27 * ws[2])),
              0.02 * rng.standard_normal(bs)]
    return np.concatenate(p).astype(np.float32)


def _adam_state(rng, n):
    """Moments and step of a training run under way."""
    return (1e-3 * rng.standard_normal(n).astype(np.float32),
            1e-6 * rng.uniform(0.5, 2.0, n).astype(np.float32), 100)


LR = 1e-3


class _Handle:
    """Owns a library handle: freed with the state that holds it."""

    def __init__(self, h, free):
        self.h, self._free = h, free

    def __del__(self):
        self._free(self.h)


def _context(case, bodies):
    flags, prec = 0, V.VIE_FP64
    if case.get("solver", "fgmres") != "fp64":
        prec = V.VIE_MIXED
    if case["body"] == "metasurface":
        flags = V.VIE_FLAG_Z_WINDOW
    opt = V.make_options(K0, precision=prec, tol=case.get("tol", 1e-11), max_iter=20000, flags=flags)
    return _Handle(V.vie_setup(bodies, opt), V.vie_destroy)


def _solve(case, ctx, chans, nrhs):
    if case.get("solver", "fgmres") == "fgmres":
        V.vie_solve_fgmres(ctx, chans, nrhs, V.fgmres_options(40, (2, 2), 8, V.VIE_MIXED_BF16))
    else:
        V.vie_solve(ctx, chans, nrhs)


def _vectors(shape, rng):
    g = torch.Generator(device="cuda").manual_seed(int(rng.integers(1 << 31)))
    return torch.complex(torch.randn(shape, generator=g, device="cuda", dtype=torch.float64),
                         torch.randn(shape, generator=g, device="cuda", dtype=torch.float64))


def _product_inputs(case, seed):
    rng = np.random.default_rng(seed)
    n = (case["nx"], case["ny"], case["nz"])
    g = Grid.centred(n, 1.0 / 32)
    r = [0.48 * m * g.h for m in n]
    x, y, z = g.mesh()
    eps = np.ones(x.shape)
    eps[(x / r[0]) ** 2 + (y / r[1]) ** 2 + (z / r[2]) ** 2 <= 1] = rng.uniform(2.0, 4.0)
    return (eps, g.h, g.origin), _vectors((case["nvec"], 3) + eps.shape, rng)


def prepare(case, seed):
    kind = case["kind"]
    rng = np.random.default_rng(seed)
    if kind == "product":
        body, x = _product_inputs(case, seed)
        ctx = _Handle(V.vie_setup([body], V.make_options(K0)), V.vie_destroy)
        return {"case": case, "ctx": ctx, "x": x, "y": torch.empty_like(x)}
    if kind == "solve":
        bodies, chans = _bodies(case, rng)
        th, ph = _directions(SCAN)
        return {"case": case, "ctx": _context(case, bodies), "chans": chans, "th": th, "ph": ph,
                "nrhs": [case["channels"]] * len(bodies)}
    if kind == "farfield":
        bodies, chans = _bodies(case, rng)
        ctx = _context(case, bodies)
        _solve(case, ctx.h, chans, [case["channels"]])
        th, ph = _directions(case)
        return {"case": case, "ctx": ctx, "th": th, "ph": ph}
    if kind.startswith("rt_"):
        eps, h, origin = _rt_body(case, rng)
        s = {"case": case, "rt": _Handle(V.vie_rt_setup(eps, h, origin, K0), V.vie_rt_destroy)}
        if kind == "rt_product":
            shape = (case["nvec"], 3) + tuple(m + 2 for m in eps.shape)
            s["x"] = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
        elif kind == "rt_solve":
            s["chans"] = [_channel(rng) for _ in range(case["channels"])]
        else:
            s["w"] = _rt_current(case, rng, eps, h, origin)
            s["th"], s["ph"] = _directions(case)
        return s
    d, feat, target, _ = _cnn_box(case, rng)
    net = _Handle(V.vie_cnn_create(0), V.vie_cnn_destroy)
    p = V.vie_cnn_params(net.h, _cnn_weights(rng))
    s = {"case": case, "net": net, "d": d, "feat": feat}
    if kind == "cnn_train":
        V.vie_cnn_adam_state(net.h, _adam_state(rng, p.size))
        s["target"] = target
    else:
        s["out"] = torch.empty(feat.shape[:3] + (16,), device="cuda")
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "product":
        V.vie_matvec_dev(s["ctx"].h, 0, s["x"].data_ptr(), s["y"].data_ptr(), case["nvec"])
        return s["y"]
    if kind == "solve":
        _solve(case, s["ctx"].h, s["chans"], s["nrhs"])
        return [V.vie_farfield(s["ctx"].h, b, s["th"], s["ph"], n) for b, n in enumerate(s["nrhs"])]
    if kind == "farfield":
        return V.vie_farfield(s["ctx"].h, 0, s["th"], s["ph"], case["channels"])
    if kind == "rt_product":
        return V.vie_rt_matvec(s["rt"].h, s["x"])
    if kind == "rt_solve":
        return V.vie_rt_solve(s["rt"].h, s["chans"], tol=case["tol"], max_iter=20000,
                              precision=V.VIE_MIXED if case["mixed"] else V.VIE_FP64)[1]
    if kind == "rt_farfield":
        return V.vie_rt_farfield(s["rt"].h, s["w"], s["th"], s["ph"])
    if kind == "cnn_infer":
        V.vie_cnn_infer_dev(s["net"].h, s["d"], s["feat"].data_ptr(), s["out"].data_ptr())
        return s["out"]
    loss = V.vie_cnn_train_step_dev(s["net"].h, s["d"], s["feat"].data_ptr(),
                                    s["target"].data_ptr(), LR)
    m, v, step = V.vie_cnn_adam_state(s["net"].h)
    return {"loss": np.float32(loss), "params": V.vie_cnn_params(s["net"].h), "m": m, "v": v,
            "step": step}


# ---------------------------------------------------------------- the work
def _pad(n):
    p = 1
    while p < 2 * n - 1:
        p *= 2
    return min(p, 3 * p // 4) if 3 * p // 4 >= 2 * n - 1 else p


def _product_work(n, nvec, fields=3, spectrum=6):
    """Vectors in and out once and the spectrum's octant once; pruned transforms there and back."""
    P = [_pad(m) for m in n]
    vox = n[0] * n[1] * n[2]
    lines = [(n[1] * n[2], P[0]), (P[0] * n[2], P[1]), (P[0] * P[1], P[2])]
    fft = 2 * fields * sum(5.0 * k * p * math.log2(p) for k, p in lines)
    octant = spectrum * (P[0] // 2 + 1) * (P[1] // 2 + 1) * (P[2] // 2 + 1) * 16
    return {"bytes": nvec * 2 * 3 * vox * 16 + vox * 8 + octant,
            "flops": nvec * (fft + 60.0 * P[0] * P[1] * P[2])}


def work(case):
    kind = case["kind"]
    if kind == "product":
        return _product_work((case["nx"], case["ny"], case["nz"]), case["nvec"])
    if kind == "solve":
        # iterations as measured on such bodies (two products each, or one per Arnoldi step)
        total = {"bytes": 0.0, "flops": 0.0}
        for b in range(case["bodies"]):
            if case["body"] == "metasurface":
                n, products = (case["n"], case["n"], 29 * case["n"] // 128), 125
            else:
                m = case["n"] * (3 if b % 2 and case["body"] == "ellipsoids" else 2) // 2
                n, products = (m, m, m), 60 if case["n"] < 20 else 300
            w = _product_work(n, case["channels"])
            for k in total:
                total[k] += products * w[k]
        return total
    if kind in ("farfield", "rt_farfield"):
        nd = case["ntheta"] * max(1, case["nphi"])
        if kind == "farfield":
            n = case["n"]
            cols, vox = n * n, 0.085 * n ** 3
        else:
            n = (case["nx"] + 2, case["ny"] + 2, case["nz"] + 2)
            cols, vox = n[0] * n[1], 0.5 * n[0] * n[1] * n[2]
        # a sum over each column per theta, then over the columns per direction
        sums = min(nd * vox, case["ntheta"] * vox + nd * cols) * 3 * case["channels"]
        return {"bytes": 48.0 * vox * case["channels"] + 32.0 * nd * case["channels"],
                "flops": 8.0 * sums}
    if kind == "rt_product":
        n = (case["nx"] + 2, case["ny"] + 2, case["nz"] + 2)
        return _product_work(n, case["nvec"], fields=3.5, spectrum=1)
    if kind == "rt_solve":
        n = (case["nx"] + 2, case["ny"] + 2, case["nz"] + 2)
        w = _product_work(n, case["channels"], fields=3.5, spectrum=1)
        return {k: 150 * v for k, v in w.items()}
    vox = float(case["d0"] * case["d1"] * case["d2"])
    flops = 2 * 27 * vox * (3 * 32 * 32 + 32 * 16)
    if kind == "cnn_infer":
        return {"bytes": vox * 128, "flops": flops}
    return {"bytes": vox * 88, "flops": flops * 3 - 2 * 27 * vox * 32 * 32}


# ------------------------------------------- the same results in plain torch
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


class _Pulse:
    """I - chi Ghat on one body's box (or the z layers that hold it) by torch FFTs in complex128."""

    def __init__(self, eps, h, origin, crop=True):
        lo, self.h = 0, h
        if crop:
            z = np.nonzero((eps != 1).any(axis=(1, 2)))[0]
            lo = z[0]
            eps = eps[lo:z[-1] + 1]
        self.n = eps.shape  # (N3, N2, N1)
        self.ax = [torch.tensor(origin[a] + h * (np.arange(self.n[2 - a]) + (lo if a == 2 else 0)),
                                device=_device()) for a in range(3)]
        self.chi = torch.tensor(eps - 1.0, device=_device())
        self.P = [2 * m for m in self.n]
        d = [torch.fft.fftfreq(p, 1.0 / p, device=_device(), dtype=torch.float64) * h for p in self.P]
        Z, Y, X = torch.meshgrid(*d, indexing="ij")
        r = torch.sqrt(X * X + Y * Y + Z * Z)
        r[0, 0, 0] = 1.0
        kr = K0 * r
        g = torch.exp(1j * kr) / (4 * math.pi * r) * (K0 * K0 * h ** 3)
        a = 1 + (1j * kr - 1) / (kr * kr)
        b = (3 - 3j * kr - kr * kr) / (kr * kr)
        x = K0 * h * (3 / (4 * math.pi)) ** (1 / 3)
        s = complex(-1 / 3 + 2 / 3 * (math.cos(x) + x * math.sin(x) - 1), (K0 * h) ** 3 / (6 * math.pi))
        R = [X / r, Y / r, Z / r]
        self.G = {}
        for i in range(3):
            for j in range(i, 3):
                t = g * (b * (R[i] * R[j]) + (a if i == j else 0))
                t[0, 0, 0] = s if i == j else 0
                self.G[i, j] = self.G[j, i] = torch.fft.fftn(t)

    def apply(self, x):  # [3][N3][N2][N1]
        f = [torch.fft.fftn(x[i], s=self.P) for i in range(3)]
        y = torch.empty_like(x)
        for i in range(3):
            c = torch.fft.ifftn(sum(self.G[i, j] * f[j] for j in range(3)))
            y[i] = x[i] - self.chi * c[: self.n[0], : self.n[1], : self.n[2]]
        return y

    def rhs(self, k, p):
        ph = [torch.exp(1j * K0 * float(k[a]) * self.ax[a]) for a in range(3)]
        e = ph[2][:, None, None] * ph[1][None, :, None] * ph[0][None, None, :]
        return torch.stack([self.chi * e * complex(p[i]) for i in range(3)])

    def farfield(self, w, th, ph):
        return _far_exact(w, self.ax, [0.0] * 3, self.h, th, ph)


def _far_exact(w, ax, half, h, th, ph):
    """F_theta, F_phi of a dense field w[3][z][y][x]; half: shift of component i's points along axis i."""
    out = torch.empty((len(th), 2), dtype=torch.complex128, device=w.device)
    t, p = (torch.tensor(v, device=w.device) for v in (th, ph))
    r = [t.sin() * p.cos(), t.sin() * p.sin(), t.cos()]
    et, ep = [t.cos() * p.cos(), t.cos() * p.sin(), -t.sin()], [-p.sin(), p.cos(), 0 * p]
    n3, n2, n1 = w.shape[1:]
    for a in range(0, len(th), 256):
        s = slice(a, min(len(th), a + 256))
        E = [torch.exp(-1j * K0 * r[i][s][:, None] * ax[i][None]) for i in range(3)]
        S = []
        for i in range(3):
            u = (w[i].reshape(n3 * n2, n1) @ E[0].T.contiguous()).reshape(n3, n2, -1)
            u = ((u * E[1].T[None]).sum(1) * E[2].T).sum(0)
            S.append(u * torch.exp(-1j * K0 * r[i][s] * half[i]))
        c = K0 * K0 * h ** 3 / (4 * math.pi)
        out[s, 0] = c * sum(et[i][s] * S[i] for i in range(3))
        out[s, 1] = c * sum(ep[i][s] * S[i] for i in range(3))
    return out


def _bicgstab(apply, b, tol=1e-13, limit=6000):
    """BiCGSTAB from zero, restarted from the true residual."""
    x, its = torch.zeros_like(b), 0
    nb = torch.linalg.vector_norm(b)
    best, stale = math.inf, 0
    while its < limit:
        r = b - apply(x)
        rel = float(torch.linalg.vector_norm(r) / nb)
        stale = stale + 1 if rel > 0.5 * best else 0
        best = min(best, rel)
        if rel <= tol or stale >= 3:
            break
        rh, p, v = r.clone(), torch.zeros_like(b), torch.zeros_like(b)
        rho = al = om = torch.ones((), dtype=b.dtype, device=b.device)
        target = max(0.5 * tol, 1e-8 * rel)
        while its < limit:
            its += 1
            rho1 = torch.vdot(rh.ravel(), r.ravel())
            p = r + (rho1 / rho) * (al / om) * (p - om * v)
            v = apply(p)
            al = rho1 / torch.vdot(rh.ravel(), v.ravel())
            s = r - al * v
            t = apply(s)
            om = torch.vdot(t.ravel(), s.ravel()) / torch.vdot(t.ravel(), t.ravel())
            x = x + al * p + om * s
            r, rho = s - om * t, rho1
            if its % 4 == 0 and float(torch.linalg.vector_norm(r) / nb) <= target:
                break
    return x


def _rt_faces(chi):
    """alpha and chi_f [3][E3][E2][E1] of the padded contrast."""
    alpha, chif = np.zeros((3,) + chi.shape), np.zeros((3,) + chi.shape)
    for i in range(3):
        up = np.roll(chi, -1, axis=2 - i)
        both, one = (chi != 0) & (up != 0), (chi != 0) ^ (up != 0)
        alpha[i] = both + 0.5 * one
        chif[i][both] = 2.0 / (1.0 / chi[both] + 1.0 / up[both])
        chif[i][one] = (chi + up)[one]
    return alpha, chif


class _Rooftop:
    """The rooftop operator by torch FFTs in complex128."""

    def __init__(self, eps, h, origin):
        chi = np.pad(eps - 1.0, 1)
        a, c = _rt_faces(chi)
        self.alpha, self.chif = torch.tensor(a, device=_device()), torch.tensor(c, device=_device())
        self.h, self.n, self.P = h, chi.shape, [2 * m for m in chi.shape]
        self.ax = [torch.tensor(origin[i] + h * (np.arange(self.n[2 - i]) - 1), device=_device())
                   for i in range(3)]
        d = [torch.fft.fftfreq(p, 1.0 / p, device=_device(), dtype=torch.float64) * h for p in self.P]
        Z, Y, X = torch.meshgrid(*d, indexing="ij")
        r = torch.sqrt(X * X + Y * Y + Z * Z)
        r[0, 0, 0] = 1.0
        g = h ** 3 * torch.exp(1j * K0 * r) / (4 * math.pi * r)
        # cube cell: radial part in closed form, one quarter face by Gauss-Legendre
        u, wt = np.polynomial.legendre.leggauss(48)
        u, wt = (u + 1) * h / 4, wt * h / 4
        R = np.sqrt(h * h / 4 + u[:, None] ** 2 + u[None] ** 2)
        f = (np.exp(1j * K0 * R) * (1 - 1j * K0 * R) - 1) / K0 ** 2 * (h / 2) / R ** 3
        g[0, 0, 0] = complex(24 * (wt[:, None] * wt[None] * f).sum() / (4 * math.pi))
        self.g = torch.fft.fftn(g)

    def _conv(self, f):
        c = torch.fft.ifftn(torch.fft.fftn(f, s=self.P) * self.g)
        return c[: self.n[0], : self.n[1], : self.n[2]]

    def apply(self, x):
        xa = x * (self.alpha > 0)
        rho = sum(xa[i] - torch.roll(xa[i], 1, dims=2 - i) for i in range(3)) / self.h
        phi = self._conv(rho)
        y = x.clone()
        for i in range(3):
            e = K0 * K0 * self._conv(self.alpha[i] * x[i]) + (torch.roll(phi, -1, dims=2 - i) - phi) / self.h
            y[i] -= self.chif[i] * e
        return y

    def rhs(self, k, p):
        b = []
        for i in range(3):
            ph = [torch.exp(1j * K0 * float(k[a]) * (self.ax[a] + (self.h / 2 if a == i else 0)))
                  for a in range(3)]
            b.append(self.chif[i] * complex(p[i]) * ph[2][:, None, None] * ph[1][None, :, None] * ph[0])
        return torch.stack(b)


def _conv3(x, W, b):
    """Same-padded 3x3x3 convolution, channels last, W[27][Cout][Cin], as 27 products."""
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    D, H, Wd, _ = x.shape
    y = b.expand(D, H, Wd, b.numel())
    for t in range(27):
        z, yy, xx = t // 9, t // 3 % 3, t % 3
        y = y + xp[z:z + D, yy:yy + H, xx:xx + Wd] @ W[t].T
    return y


def _cnn_exact(p, feat):
    layers, at, x = [], 0, feat.double()
    for ws, bs in CNN_SHAPES:
        n = int(np.prod(ws))
        layers.append((p[at:at + n].reshape(ws), p[at + n:at + n + bs[0]]))
        at += n + bs[0]
    for k, (W, b) in enumerate(layers):
        x = _conv3(x, W, b)
        if k + 1 < len(layers):
            x = torch.relu(x)
    return x


def exact(case, seed):
    kind = case["kind"]
    rng = np.random.default_rng(seed)
    if kind == "product":
        body, x = _product_inputs(case, seed)
        op = _Pulse(*body, crop=False)  # x acts from every layer
        return torch.stack([op.apply(v) for v in x])
    if kind in ("solve", "farfield"):
        bodies, chans = _bodies(case, rng)
        th, ph = _directions(case if kind == "farfield" else SCAN)
        out = []
        for b, body in enumerate(bodies):
            if b > 0 and case["body"] != "sphere":
                out.append(None)  # one body of a batch: each further one takes as long
                continue
            op = _Pulse(*body)
            F = [op.farfield(_bicgstab(op.apply, op.rhs(*c)), th, ph)
                 for c in chans[b * case["channels"]:(b + 1) * case["channels"]]]
            out.append(torch.stack(F))
        return out if kind == "solve" else out[0]
    if kind.startswith("rt_"):
        eps, h, origin = _rt_body(case, rng)
        op = _Rooftop(eps, h, origin)
        if kind == "rt_product":
            shape = (case["nvec"], 3) + tuple(m + 2 for m in eps.shape)
            x = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
            return torch.stack([op.apply(torch.tensor(v, device=_device())) for v in x])
        if kind == "rt_solve":
            chans = [_channel(rng) for _ in range(case["channels"])]
            return torch.stack([_bicgstab(op.apply, op.rhs(*c)) for c in chans])
        w = torch.tensor(_rt_current(case, rng, eps, h, origin), device=_device())
        th, ph = _directions(case)
        return torch.stack([_far_exact(op.alpha * v, op.ax, [h / 2] * 3, h, th, ph) for v in w])
    d, feat, target, body = _cnn_box(case, rng)
    p = torch.tensor(_cnn_weights(rng), device="cuda").double().requires_grad_(kind == "cnn_train")
    out = _cnn_exact(p, feat)
    if kind == "cnn_infer":
        return out
    t = target.double()
    loss = (((out[..., :6] - t) * body[..., None]) ** 2).sum() / (t ** 2).sum()
    (g,) = torch.autograd.grad(loss, p)
    m, v, step = _adam_state(rng, p.numel())
    m = 0.9 * torch.tensor(m, device="cuda").double() + 0.1 * g
    v = 0.999 * torch.tensor(v, device="cuda").double() + 0.001 * g * g
    step += 1
    q = p.detach() - LR * (m / (1 - 0.9 ** step)) / (torch.sqrt(v / (1 - 0.999 ** step)) + 1e-8)
    return {"loss": float(loss), "params": q, "m": m, "v": v, "step": None}
