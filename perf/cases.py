"""The work that programs built on this library have it do, as timed cases.

``listed()`` names the cases, ``draw(rng)`` makes more of the same ranges,
``prepare`` builds what a program holds before the call (plan, tiling, network,
measurements on the GPU), ``run`` is one pass through the public entry points
and ``exact`` the same result in 64 bits by plain torch.

Kinds of pass:
  apply   y = A x and g = A^H r on one plan (the two calls that every solver,
          power iteration and custom reconstruction is made of)
  fista   one FISTA reconstruction of `iters` iterations from zero
  batch   one replay of a persistent batch of uneven scans
  net     one inference of the learned unrolled network
  grad    one gradient of its training loss
Geometry and pulse are those of the package's workloads (5900 m/s, 40 MHz
sampling, 4 MHz Gabor pulse, 0.5 mm pitch) or of the 50 x 50 x 50 simulated
specimen (``sim``).  Bins, beam and signs belong to the plan and follow from the
case; scenes, noise and operands follow from the seed.
"""
import collections
import math
import os

import numpy as np
import torch

import paper_2012_04534_amd as pkg
from paper_2012_04534_amd import ufss

PKG = os.path.dirname(os.path.abspath(pkg.__file__))
MU = 0.1


def _case(name, kind, nx, ny, nz, nt, m, algo, **over):
    c = dict(name=name, kind=kind, nx=nx, ny=ny, nz=nz, nt=nt, m=m, algo=algo, dtype="f32",
             per_position=False, win=-1, sim=False, mixed=False, tuned=False, iters=1, stages=0,
             scans=0, bins_seed=1)
    c.update(over)
    return c


def listed():
    return [
        # the smallest reconstruction: one 32-position B-scan, launches and latency count
        _case("bscan32_fista", "fista", 32, 1, 128, 256, 32, "gemm", iters=20, bins_seed=1001),
        # the default operator on the 32 x 32 C-scan with its own 64 bins per
        # position, tiling from the shipped cache: the benchmark's FISTA step
        _case("cscan32_fista", "fista", 32, 32, 256, 512, 64, "gemm", per_position=True, tuned=True,
              iters=3, bins_seed=1002),
        # the largest ordinary C-scan, windowed aperture, FP32 products
        _case("cscan64_apply", "apply", 64, 64, 512, 1024, 128, "gemm", win=16, tuned=True,
              bins_seed=1003),
        # the same scan with BF16 operands, for users who trade accuracy for time
        _case("cscan64_apply_bf16", "apply", 64, 64, 512, 1024, 128, "gemm", dtype="bf16", win=16,
              tuned=True, bins_seed=1003),
        # the transform operator: the fastest way to a 32 x 32 reconstruction
        _case("cscan32_fista_transform", "fista", 32, 32, 256, 512, 64, "fft", per_position=True,
              iters=20, bins_seed=1002),
        # the transform operator where its table is far larger than the caches
        _case("cscan64_apply_transform", "apply", 64, 64, 512, 1024, 128, "fft", win=16, bins_seed=1003),
        # an uneven grid with nothing a multiple of a tile, BF16 table
        _case("cscan45x51_apply_transform_bf16", "apply", 45, 51, 301, 602, 75, "fft", dtype="bf16",
              win=16, per_position=True, bins_seed=1005),
        # few bins per position with the Gaussian beam (the simulated specimen, n_f = 2)
        _case("sim50_apply_few_bins", "apply", 50, 50, 50, 256, 2, "auto", per_position=True, sim=True,
              bins_seed=5001),
        # randomly mixed measurements of the same specimen (n_f = 10, signs per position)
        _case("sim50_apply_mixed", "apply", 50, 50, 50, 256, 10, "fft", per_position=True, sim=True,
              mixed=True, bins_seed=5002),
        # several uneven scans reconstructed together (B- and C-scans, default tilings)
        _case("batch_uneven", "batch", 48, 48, 320, 640, 83, "gemm", win=16, scans=8, iters=5, bins_seed=1004),
        # learned reconstruction of the 32 x 32 C-scan with the shipped network
        _case("cscan32_net", "net", 32, 32, 256, 512, 64, "fft", per_position=True, stages=16, bins_seed=1002),
        # one training gradient (forward and backward) of a network's first stages
        _case("cscan32_net_grad", "grad", 32, 32, 256, 512, 64, "fft", per_position=True, stages=4,
              bins_seed=1002),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# the listed cases' largest pass, in complex products of the windowed sum
_MOST_PRODUCTS = 2 * 64 * 64 * 512 * 128 * 28.8 ** 2


def draw(rng):
    while True:
        c = _case("", "apply", 32, 1, 128, 256, 32, "gemm", bins_seed=rng.randrange(1 << 20))
        del c["name"]
        what = rng.choice(["gemm", "gemm", "gemm", "bf16", "fft", "fft", "fft_bf16", "few", "mixed", "batch",
                           "net", "grad"])
        c["nx"] = _log_int(rng, 16, 64)
        c["ny"] = 1 if rng.random() < 0.3 else _log_int(rng, 16, 64)
        c["nz"] = _log_int(rng, 48, 512)
        c["nt"] = 2 * c["nz"] if rng.random() < 0.5 else 1 << max(7, (2 * c["nz"] - 1).bit_length())
        c["win"] = 16 if c["ny"] > 1 and rng.random() < 0.6 else -1
        c["per_position"] = rng.random() < 0.5
        if what in ("few", "mixed"):
            c.update(sim=True, nx=_log_int(rng, 16, 50), ny=_log_int(rng, 16, 50), nz=_log_int(rng, 24, 100),
                     nt=256, win=-1, per_position=True, m=rng.choice([1, 2, 5]))
            if what == "few":
                c["algo"] = "auto"
            else:
                c.update(algo="fft", mixed=True, per_position=rng.random() < 0.5, m=_log_int(rng, 1, 20))
            if c["nx"] * c["ny"] * c["nz"] > 50 ** 3:
                continue
        else:
            band = len(_band(_geometry(c)))
            if band < 8:
                continue
            c["m"] = min(band, _log_int(rng, 8, 128))
            if what == "batch":
                c.update(kind="batch", algo="gemm", nx=48, ny=48, nz=_log_int(rng, 64, 320), win=16, m=1,
                         scans=rng.randint(2, 8), iters=rng.randint(2, 5))
                c["nt"] = 2 * c["nz"]
            else:
                c["algo"] = "fft" if what in ("fft", "fft_bf16", "net", "grad") else "gemm"
                c["dtype"] = "bf16" if what in ("bf16", "fft_bf16") else "f32"
                if what in ("net", "grad"):
                    c.update(kind=what, stages=rng.randint(1, 4))
                elif c["dtype"] == "f32" and rng.random() < 0.4:
                    c.update(kind="fista", iters=rng.randint(1, 8))
        if c["kind"] != "batch":
            passes = {"fista": 2 * c["iters"] + 1, "net": 2 * c["stages"] + 1, "grad": 4 * c["stages"] + 1}
            p = _window_products(c, False) * passes.get(c["kind"], 2)
            if p * (4 if what == "few" else 1) > _MOST_PRODUCTS or c["nx"] * c["ny"] * c["nz"] > 64 * 64 * 512:
                continue
            if what in ("net", "grad") and c["nx"] * c["ny"] * c["nz"] > 32 * 32 * 256:
                continue
        return c


# ---------------------------------------------------------------------------
# Geometry, pulse and bins (plain numpy).
# ---------------------------------------------------------------------------
def _geometry(c):
    if c["sim"]:
        bw = 2.0 * math.sqrt(2.0 * math.log(2.0)) * 0.65 * math.sqrt(2.0) / (2.0 * math.pi)
        return dict(nx=c["nx"], ny=c["ny"], nz=c["nz"], nt=c["nt"], dx=0.5e-3, dy=0.5e-3, dz=5920.0 / 40e6,
                    z_start=29.6e-3, t0=10e-6, c=5920.0, fs=20e6, fc=3.2e6, frac_bw=bw, band_db=40.0,
                    win_x=c["win"], win_y=c["win"], theta=math.radians(30.0))
    return dict(nx=c["nx"], ny=c["ny"], nz=c["nz"], nt=c["nt"], dx=0.5e-3, dy=0.5e-3, dz=73.75e-6,
                z_start=29.6e-3, t0=float("nan"), c=5900.0, fs=40e6, fc=4e6, frac_bw=0.5, band_db=40.0,
                win_x=c["win"], win_y=c["win"], theta=0.0)


def _sigma_f(g):
    return g["frac_bw"] * g["fc"] / (2.0 * math.sqrt(2.0 * math.log(2.0)))


def _spectrum(g, k):
    sf = _sigma_f(g)
    f = np.asarray(k, dtype=np.float64) * g["fs"] / g["nt"]
    return g["fs"] * math.sqrt(2.0 * math.pi) / (2.0 * math.pi * sf) * np.exp(-(f - g["fc"]) ** 2 / (2.0 * sf * sf))


def _band(g):
    k = np.arange(g["nt"] // 2 + 1)
    env = np.exp(-(k * g["fs"] / g["nt"] - g["fc"]) ** 2 / (2.0 * _sigma_f(g) ** 2))
    return k[env >= 10.0 ** (-g["band_db"] / 20.0)]


def _window(g):
    full = lambda n, w: n - 1 if w < 0 else min(w, n - 1)
    return full(g["nx"], g["win_x"]), full(g["ny"], g["win_y"])


def _bins_and_signs(c, g):
    rng = np.random.default_rng(c["bins_seed"])
    pool = np.arange(g["nt"]) if c["mixed"] else _band(g)
    rows = g["nx"] * g["ny"] if c["per_position"] else 1
    pick = np.argsort(rng.random((rows, len(pool))), axis=1)[:, :c["m"]]
    bins = np.sort(pool[pick], axis=1).astype(np.int32)
    bins = bins.reshape(g["ny"], g["nx"], c["m"]) if c["per_position"] else bins.reshape(c["m"])
    signs = None
    if c["mixed"]:
        signs = (2 * rng.integers(0, 2, size=(g["ny"], g["nx"], g["nt"])) - 1).astype(np.int8)
    return bins, signs


def _scans(c):
    """The single-scan cases of a batch: lateral 16..nx, depth 64..nz, half of them B-scans."""
    if c["kind"] != "batch":
        return [c]
    rng = np.random.default_rng(c["bins_seed"])
    out = []
    for i in range(c["scans"]):
        s = dict(c, kind="fista", nx=int(rng.integers(16, c["nx"] + 1)), nz=int(rng.integers(64, c["nz"] + 1)),
                 ny=int(rng.integers(16, c["ny"] + 1)) if i % 2 else 1, bins_seed=c["bins_seed"] + 1 + i,
                 per_position=bool(rng.integers(2)))
        s["nt"] = 2 * s["nz"]
        s["win"] = 16 if s["ny"] > 1 else -1
        band = len(_band(_geometry(s)))
        s["m"] = int(rng.integers(max(1, band // 2), band + 1))
        out.append(s)
    return out


# ---------------------------------------------------------------------------
# The operator in 64 bits: a cyclic lateral correlation of length N + W per
# axis, its phasors from the closed form.
# ---------------------------------------------------------------------------
def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


class Operator64:
    def __init__(self, c):
        g = _geometry(c)
        self.g, dev = g, _dev()
        nx, ny, nz, nt = g["nx"], g["ny"], g["nz"], g["nt"]
        wx, wy = _window(g)
        self.lx, self.ly = nx + wx, ny + wy
        bins, signs = _bins_and_signs(c, g)
        flat = bins.reshape(-1, c["m"])
        if c["mixed"]:
            self.ubins = np.where(np.arange(nt) <= nt // 2, np.arange(nt), np.arange(nt) - nt)
        else:
            self.ubins = np.unique(flat)
        mu = len(self.ubins)
        t64 = dict(dtype=torch.float64, device=dev)
        delay = lambda x, y, z: (2.0 / g["c"]) * torch.sqrt(x * x + y * y + z * z)
        z = g["z_start"] + g["dz"] * torch.arange(nz, **t64)
        t0 = g["t0"]
        if math.isnan(t0):
            far = math.sqrt((wx * g["dx"]) ** 2 + (wy * g["dy"]) ** 2 + float(z[-1]) ** 2)
            t0 = 0.5 * (2.0 / g["c"]) * (g["z_start"] + far) - nt / (2.0 * g["fs"])
        ax = g["dx"] * torch.arange(wx + 1, **t64)[None, :, None]
        ay = g["dy"] * torch.arange(wy + 1, **t64)[:, None, None]
        turns = (delay(ax, ay, z) - t0) * g["fs"] / nt
        k = torch.tensor(self.ubins, **t64)
        ph = torch.remainder(turns[..., None] * k, 1.0) * (-2.0 * math.pi)
        amp = torch.ones_like(turns)
        if g["theta"] > 0:
            amp = torch.exp(-(ax * ax + ay * ay) / (z * math.tan(g["theta"])) ** 2)
        P = torch.stack([amp[..., None] * torch.cos(ph), amp[..., None] * torch.sin(ph)], dim=-1)
        del ph

        def weights(length, w):
            q = torch.arange(length // 2 + 1, **t64)[:, None]
            d = torch.arange(w + 1, **t64)[None, :]
            return torch.where(d == 0, 1.0, 2.0) * torch.cos(2.0 * math.pi * torch.remainder(q * d, length) / length)

        K = torch.matmul(weights(self.lx, wx), P.reshape(wy + 1, wx + 1, -1))
        del P
        K = torch.matmul(weights(self.ly, wy), K.reshape(wy + 1, -1))
        self.K = torch.view_as_complex(K.reshape(self.ly // 2 + 1, self.lx // 2 + 1, nz, mu, 2))

        def dft(rows, cols, length, sign):
            a = torch.remainder(torch.arange(rows, **t64)[:, None] * torch.arange(cols, **t64)[None, :], length)
            return torch.polar(torch.ones_like(a), sign * 2.0 * math.pi * a / length)

        self.fx, self.fy = dft(self.lx, nx, self.lx, -1.0), dft(self.ly, ny, self.ly, -1.0)
        self.ix, self.iy = dft(nx, self.lx, self.lx, 1.0) / self.lx, dft(ny, self.ly, self.ly, 1.0) / self.ly
        self.ox = torch.tensor([min(q, self.lx - q) for q in range(self.lx)], device=dev)
        self.oy = [min(q, self.ly - q) for q in range(self.ly)]
        self.h = torch.tensor(_spectrum(g, self.ubins), **t64)
        npos = nx * ny
        self.mix = None
        if c["mixed"]:
            xi = torch.fft.fft(torch.tensor(signs.reshape(npos, nt), dtype=torch.complex128), dim=-1).to(dev) / nt
            kb = torch.tensor(np.broadcast_to(flat, (npos, c["m"])).copy(), device=dev).long()
            at = torch.remainder(kb[:, :, None] - torch.arange(nt, device=dev), nt)
            self.mix = torch.gather(xi[:, None, :].expand(npos, c["m"], nt), 2, at)
        else:
            at = np.searchsorted(self.ubins, np.broadcast_to(flat, (npos, c["m"])))
            self.at = torch.tensor(at, device=dev).long()
        self._L = None

    def _lateral(self, W_y, W_x, v):
        v = torch.matmul(W_x, v)
        return torch.matmul(W_y, v.reshape(v.shape[0], -1)).reshape(W_y.shape[0], v.shape[1], v.shape[2])

    def forward(self, x):
        """[ny, nx, nz] complex128 -> [ny nx, m]"""
        g = self.g
        X = self._lateral(self.fy, self.fx, x)
        Y = torch.stack([(self.K[self.oy[q]][self.ox] * X[q][:, :, None]).sum(1) for q in range(self.ly)])
        y = self._lateral(self.iy, self.ix, Y).reshape(g["nx"] * g["ny"], -1) * self.h
        if self.mix is not None:
            return (self.mix * y[:, None, :]).sum(-1)
        return torch.gather(y, 1, self.at)

    def adjoint(self, r):
        """[ny nx, m] complex128 -> [ny, nx, nz]"""
        g = self.g
        if self.mix is not None:
            R = (self.mix.conj() * r[:, :, None]).sum(1)
        else:
            R = torch.zeros(r.shape[0], len(self.ubins), dtype=r.dtype, device=r.device)
            R.scatter_(1, self.at, r)
        R = self._lateral(self.fy, self.fx, (R * self.h).reshape(g["ny"], g["nx"], -1))
        X = torch.stack([(self.K[self.oy[q]][self.ox].conj() * R[q][:, None, :]).sum(-1) for q in range(self.ly)])
        return self._lateral(self.iy, self.ix, X)

    def lipschitz(self):
        """A power-iteration quotient with a margin, as a program sets the step."""
        if self._L is None:
            g = self.g
            v = torch.randn(g["ny"], g["nx"], g["nz"], dtype=torch.complex128,
                            generator=torch.Generator().manual_seed(4)).to(_dev())
            for _ in range(12):
                v = v / torch.linalg.vector_norm(v)
                y = self.forward(v)
                v = self.adjoint(y)
            self._L = 1.3 * float(y.abs().square().sum())
        return self._L


_OPS = collections.OrderedDict()


def _operator(c):
    key = tuple(sorted((k, v) for k, v in c.items() if k in ("nx", "ny", "nz", "nt", "m", "per_position", "win", "sim",
                                                            "mixed", "bins_seed")))
    if key not in _OPS:
        _OPS[key] = Operator64(c)
    _OPS.move_to_end(key)
    while len(_OPS) > 8:
        _OPS.popitem(last=False)
    return _OPS[key]


# ---------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------
def _randn(shape, seed):
    return torch.randn(shape, dtype=torch.complex64, generator=torch.Generator().manual_seed(seed)).to(_dev())


def _measurements(c, seed):
    """(scene, measurements) of point scatterers, half the time over a back wall, with noise."""
    op, g = _operator(c), _geometry(c)
    rng = np.random.default_rng(seed)
    x = torch.zeros(g["ny"], g["nx"], g["nz"], dtype=torch.complex128)
    n = int(rng.integers(5, 51))
    iz = rng.integers(0, max(1, g["nz"] - 24), n)
    x[rng.integers(0, g["ny"], n), rng.integers(0, g["nx"], n), iz] = torch.tensor(rng.uniform(0.5, 1.0, n) + 0j)
    if rng.integers(2):
        x[:, :, g["nz"] - 16] = 1.0
    x = x.to(_dev())
    y = op.forward(x)
    snr = 10.0 ** (rng.uniform(10.0, 25.0) / 10.0)
    s = torch.sqrt(y.abs().square().mean() / snr)
    y = y + s * torch.randn(y.shape, dtype=torch.complex128, generator=torch.Generator().manual_seed(seed + 1)).to(_dev())
    return x.to(torch.complex64), y.to(torch.complex64)


def _net_params(c, seed):
    """The shipped network's parameters (the first stages of it)."""
    with open(os.path.join(PKG, "weights", "unrolled_cscan32_s16c8.bin"), "rb") as f:
        f.seek(8 + 8 + 16 + 8)
        p = np.frombuffer(f.read(), dtype="<f4")
    return p[:c["stages"] * (len(p) // 3 // 16)].copy()


def _plan(c):
    g = _geometry(c)
    bins, signs = _bins_and_signs(c, g)
    algo = {"auto": ufss.ALGO_AUTO, "gemm": ufss.ALGO_GEMM, "fft": ufss.ALGO_FFT}[c["algo"]]
    plan = ufss.Plan(g, c["m"], c["per_position"], bins, dtype=ufss.BF16 if c["dtype"] == "bf16" else ufss.F32,
                     algo=algo, signs=signs)
    if c["tuned"]:
        ufss.ufss_autotune(plan, cache_path=os.path.join(PKG, "tuning_gfx950.json"), use_cache=True, write_cache=False)
    return plan


def _empty_x(c):
    return torch.zeros(c["ny"], c["nx"], c["nz"], dtype=torch.complex64, device=_dev())


def prepare(case, seed):
    c = case
    if c["kind"] == "apply":
        return dict(c=c, plan=_plan(c), x=_randn((c["ny"], c["nx"], c["nz"]), seed),
                    r=_randn((c["nx"] * c["ny"], c["m"]), seed + 1),
                    y=torch.empty(c["nx"] * c["ny"], c["m"], dtype=torch.complex64, device=_dev()), g=_empty_x(c))
    if c["kind"] == "fista":
        return dict(c=c, plan=_plan(c), y=_measurements(c, seed)[1], L=_operator(c).lipschitz(), x=_empty_x(c))
    if c["kind"] == "batch":
        scans = _scans(c)
        ys = [_measurements(s, seed + 2 * i)[1] for i, s in enumerate(scans)]
        xs = [_empty_x(s) for s in scans]
        batch = ufss.Batch([_plan(s) for s in scans], ys, xs, [ufss.lambda_from_mu(MU)] * len(scans),
                           [_operator(s).lipschitz() for s in scans], c["iters"])
        return dict(c=c, batch=batch, xs=xs)
    x, y = _measurements(c, seed)
    net = ufss.Net(_plan(c), stages=c["stages"], channels=8, L=_operator(c).lipschitz(), mu=MU)
    ufss.ufss_unrolled_params(net, set_to=_net_params(c, seed))
    return dict(c=c, net=net, y=y, x=_empty_x(c), target=x)


def run(state):
    c = state["c"]
    if c["kind"] == "apply":
        ufss.ufss_forward(state["plan"], state["x"], state["y"])
        ufss.ufss_adjoint(state["plan"], state["r"], state["g"])
        return state["y"], state["g"]
    if c["kind"] == "fista":
        state["x"].zero_()
        st = ufss.ufss_fista(state["plan"], state["y"], ufss.lambda_from_mu(MU), state["L"], c["iters"], state["x"])
        # FP64 sums of FP32 iterates: FP32 holds their digits
        return dict(x=state["x"], obj=st["obj"].astype(np.float32), res=st["res"].astype(np.float32))
    if c["kind"] == "batch":
        for x in state["xs"]:
            x.zero_()
        res, _ = state["batch"].run()
        return dict(xs=state["xs"], res=res.astype(np.float32))
    if c["kind"] == "net":
        ufss.ufss_unrolled_forward(state["net"], state["y"], state["x"])
        return state["x"]
    loss, grad = ufss.ufss_unrolled_grad(state["net"], state["y"], state["target"])
    return dict(loss=loss, grad=grad)


# ---------------------------------------------------------------------------
# What a pass cannot do without.
# ---------------------------------------------------------------------------
def _window_products(c, folded):
    """Complex products of one apply of the windowed sum; folded: voxels at
    mirrored lateral offsets of a position share one phasor and one product."""
    g = _geometry(c)
    wx, wy = _window(g)

    def axis(n, w):
        if folded:
            return sum(max(min(p, w), min(n - 1 - p, w)) + 1 for p in range(n))
        return sum(min(p, w) + min(n - 1 - p, w) + 1 for p in range(n))

    per = c["m"] if not c["mixed"] else g["nt"]
    return axis(g["nx"], wx) * axis(g["ny"], wy) * g["nz"] * per


def _apply_work(c):
    """(bytes, flops) of one forward or adjoint apply."""
    g = _geometry(c)
    nvox, nmeas = g["nx"] * g["ny"] * g["nz"], g["nx"] * g["ny"] * c["m"]
    io = 8.0 * (nvox + nmeas)
    if c["algo"] != "fft":
        return io, 8.0 * _window_products(c, True)
    wx, wy = _window(g)
    lx, ly = g["nx"] + wx, g["ny"] + wy
    mu = g["nt"] if c["mixed"] else min(len(_band(g)), c["m"] * g["nx"] * g["ny"])
    # the distinct entries of the transformed kernel, even along both axes and
    # symmetric in them where the axes are alike
    nox, noy = lx // 2 + 1, ly // 2 + 1
    entries = nox * (nox + 1) // 2 if (nox == noy and lx == ly) else nox * noy
    table = entries * g["nz"] * mu * (4.0 if c["dtype"] == "bf16" else 8.0)
    return io + table, 8.0 * lx * ly * g["nz"] * mu


def work(case):
    byts = flops = 0.0
    for s in _scans(case):
        b, f = _apply_work(s)
        n = {"apply": 2, "fista": 2 * s["iters"] + 1, "net": 2 * s["stages"] + 1, "grad": 4 * s["stages"] + 1}[s["kind"]]
        nvox = s["nx"] * s["ny"] * s["nz"]
        if s["kind"] == "fista":          # the iterate and its extrapolation, read and written per iteration
            byts += s["iters"] * 32.0 * nvox
        if s["kind"] in ("net", "grad"):  # two convolutions of 2 x 8 channels x 27 taps per stage
            conv = 2.0 * 2 * 2 * 8 * 27 * nvox * s["stages"]
            flops += conv * (3 if s["kind"] == "grad" else 1)
            byts += s["stages"] * nvox * (2 * 32.0 + 40.0) * (3 if s["kind"] == "grad" else 1)
        if case["kind"] == "batch":       # the threshold rule is resolved when the batch is made
            n -= 1
        byts += n * b
        flops += n * f
    return {"bytes": byts, "flops": flops}


# ---------------------------------------------------------------------------
# The same results in 64 bits.
# ---------------------------------------------------------------------------
def _soft(z, t):
    mag = z.abs()
    return torch.where(mag > t, z * (1.0 - t / mag.clamp_min(1e-300)), torch.zeros_like(z))


def _fista64(c, y, L):
    op = _operator(c)
    y = y.to(torch.complex128)
    lam = MU * float(op.adjoint(y).abs().max())
    x = torch.zeros(c["ny"], c["nx"], c["nz"], dtype=torch.complex128, device=y.device)
    gam, t, obj, res = x, 1.0, [], []
    for _ in range(c["iters"]):
        r = op.forward(gam) - y
        r2 = float(r.abs().square().sum())
        obj.append(0.5 * r2 + lam * float(gam.abs().sum()))
        res.append(math.sqrt(r2))
        new = _soft(gam - op.adjoint(r) / L, lam / L)
        tn = 0.5 * (1.0 + math.sqrt(1.0 + 4.0 * t * t))
        gam, x, t = new + ((t - 1.0) / tn) * (new - x), new, tn
    return x, np.array(obj), np.array(res)


class _Apply(torch.autograd.Function):
    @staticmethod
    def forward(ctx, v, op):
        ctx.op = op
        return op.forward(v)

    @staticmethod
    def backward(ctx, gr):
        return ctx.op.adjoint(gr), None


class _ApplyT(torch.autograd.Function):
    @staticmethod
    def forward(ctx, v, op):
        ctx.op = op
        return op.adjoint(v)

    @staticmethod
    def backward(ctx, gr):
        return ctx.op.forward(gr), None


def _conv64(W, b, v):
    """3 x 3 x 3 convolution, zero padding: W [o, c, 27], v [c, ny, nx, nz]."""
    _, ny, nx, nz = v.shape
    p = torch.nn.functional.pad(v, (1, 1, 1, 1, 1, 1))
    out = b[:, None].expand(-1, ny * nx * nz)
    for e in range(27):
        ey, ex, ez = e // 9, (e // 3) % 3, e % 3
        out = out + torch.matmul(W[:, :, e], p[:, ey:ey + ny, ex:ex + nx, ez:ez + nz].reshape(v.shape[0], -1))
    return out.reshape(-1, ny, nx, nz)


def _net64(c, y, params, L):
    op, ch = _operator(c), 8
    y = y.to(torch.complex128)
    lam = MU * float(op.adjoint(y).abs().max())
    scale = lam / L
    x = xp = torch.zeros(c["ny"], c["nx"], c["nz"], dtype=torch.complex128, device=y.device)
    t = 1.0
    for i, p in enumerate(params.reshape(c["stages"], -1)):
        beta = 0.0
        if i > 0:
            tn = 0.5 * (1.0 + math.sqrt(1.0 + 4.0 * t * t))
            beta, t = (t - 1.0) / tn, tn
        gam = x + beta * (x - xp)
        z = gam - (torch.exp(p[0]) / L) * _ApplyT.apply(_Apply.apply(gam, op) - y, op)
        th = torch.exp(p[1]) * scale
        mag = z.abs()
        on = mag > th
        u = torch.where(on, z * (1.0 - th / torch.where(on, mag, torch.ones_like(mag))), torch.zeros_like(z))
        o = 2
        W1, o = p[o:o + ch * 54].reshape(ch, 2, 27), o + ch * 54
        b1, o = p[o:o + ch], o + ch
        W2, o = p[o:o + ch * 54].reshape(2, ch, 27), o + ch * 54
        h = torch.relu(_conv64(W1, b1, torch.stack([u.real, u.imag]) / scale))
        v = scale * _conv64(W2, p[o:o + 2], h)
        xp, x = x, u + torch.complex(v[0], v[1])
    return x


def exact(case, seed):
    c = case
    if c["kind"] == "apply":
        op = _operator(c)
        x = _randn((c["ny"], c["nx"], c["nz"]), seed).to(torch.complex128)
        r = _randn((c["nx"] * c["ny"], c["m"]), seed + 1).to(torch.complex128)
        return op.forward(x), op.adjoint(r)
    if c["kind"] == "fista":
        x, obj, res = _fista64(c, _measurements(c, seed)[1], _operator(c).lipschitz())
        return dict(x=x, obj=obj, res=res)
    if c["kind"] == "batch":
        got = [_fista64(s, _measurements(s, seed + 2 * i)[1], _operator(s).lipschitz())
               for i, s in enumerate(_scans(c))]
        return dict(xs=[v[0] for v in got], res=np.array([v[2][-1] for v in got]))
    x, y = _measurements(c, seed)
    p = torch.tensor(_net_params(c, seed), dtype=torch.float64, device=_dev())
    L = _operator(c).lipschitz()
    if c["kind"] == "net":
        with torch.no_grad():
            return _net64(c, y, p, L)
    p.requires_grad_(True)
    target = x.to(torch.complex128)
    loss = (_net64(c, y, p, L) - target).abs().square().sum() / target.abs().square().sum()
    loss.backward()
    return dict(loss=float(loss.detach()), grad=p.grad.detach())
