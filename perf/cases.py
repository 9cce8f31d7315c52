"""Workloads of the SFT inner-product library that its speed is measured on.

A case names a path (``kind``) and its sizes; ``prepare`` makes what a program has in hand before
the call (data handle, bank, network, strain), ``run`` makes one pass through the public entry
points, ``exact`` gives the same outputs from plain torch in 64 bits, ``work`` the bytes and
operations that the path cannot do without.

Kinds
  ip     one template, host in and host out (the smallest call: follow-up of a candidate)
  bank   a template-bank scan; ``data`` chooses the data set:
           ground  up to three detectors, SFTs of 32 s at 128 Hz, 5% gaps, band [32, 512), K = 8
                   (form "plain", "fstat": the F-statistic, "doppler": sky positions, one
                   waveform per detector, with the F-statistic)
           space   one detector, 60 SFTs of 2 days, wide drift, ragged ranges, K = 32
           bns     one detector, SFTs of 73 s at 40 Hz, every bin stored, K = 50
           tiny    one detector, SFTs of 64 s at 32 Hz, K = 4 Dirichlet, FP64 or FP32 sums
  sfts   SFTs and their noise estimate from raw strain (segments of a power of two), or of any
         even length with a known white noise level
  infer  the surrogate network and its derivative
  train  mini-batch training of the surrogate network
  sur    a bank scan with the surrogate waveform
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2502_11823_amd import sft

TSUN = 4.925490947641267e-6
DAY = 86400.0
YEAR = 3.15576e7
DEV = "cuda"
SITES = ((0.81, -1.58), (0.53, -2.08), (0.76, 0.18))   # latitude, longitude of three detectors
SUR = dict(mc=(1.19, 1.21), q=(1.0, 2.0), ln_tau=(math.log(600.0), math.log(16984.0)), c_phi=2.0, c_amp=0.01)


# ------------------------------------------------------------------------------------- cases
def listed():
    return [
        # one candidate followed up on a day and a half of three-detector data: latency
        dict(name="ip-ground", kind="ip", n_slots=4096, n_det=3, K=8),
        # a thousand templates around a candidate on the same data
        dict(name="bank-ground-1k", kind="bank", data="ground", form="plain", n=1000, n_slots=4096, n_det=3, K=8),
        # the benchmark's bank: the search itself
        dict(name="bank-ground-100k", kind="bank", data="ground", form="plain", n=100000, n_slots=4096, n_det=3, K=8),
        # a targeted search with sky positions: Doppler form with the F-statistic
        dict(name="bank-doppler-20k", kind="bank", data="ground", form="doppler", n=20000, n_slots=4096, n_det=3, K=8),
        # massive binaries in a space-based detector
        dict(name="bank-space-200k", kind="bank", data="space", form="plain", n=200000, n_slots=60, n_det=1, K=32),
        # the batch of a thousand waveforms of the paper's neutron-star timing
        dict(name="bank-bns-1k", kind="bank", data="bns", form="plain", n=1000, n_slots=6384, n_det=1, K=50),
        # 3.5PN templates in the FP64 reference arithmetic (an odd count)
        dict(name="bank-pn35-f64-30k", kind="bank", data="tiny", form="plain", n=30001, n_slots=256, n_det=1, K=4,
             waveform="pn35", precision="fp64"),
        # the three-detector data set from raw strain
        dict(name="sfts-ground", kind="sfts", n_samples=4096, n_seg=4096, n_det=3, w=25),
        # the accuracy study's segments: 106 s at 40 Hz (not a power of two), 129 h of data
        dict(name="sfts-study", kind="sfts", n_samples=4240, n_seg=4396, n_det=1, w=0),
        # the surrogate network alone, in its default FP64 arithmetic
        dict(name="infer-f64-1m", kind="infer", mode="fp64", hidden=128, layers=4, n=1 << 20),
        # 32 steps of training with the batch of the benchmark's surrogate
        dict(name="train-b4096", kind="train", hidden=128, layers=4, batch=4096, steps=32),
        # a surrogate bank in the split BF16 arithmetic
        dict(name="sur-scan-32k", kind="sur", mode="bf16x3", hidden=128, layers=4, n=32768, n_slots=256, K=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("ip", "bank", "bank", "bank", "bank", "bank", "sfts", "sfts", "infer", "train", "sur"))
    if kind == "ip":
        return dict(kind=kind, n_slots=_log(rng, 200, 4096), n_det=rng.randint(1, 3), K=rng.choice((4, 8, 8, 12, 16)))
    if kind == "bank":
        data = rng.choice(("ground", "ground", "space", "bns", "tiny"))
        if data == "ground":
            form = rng.choice(("plain", "plain", "fstat", "doppler"))
            return dict(kind=kind, data=data, form=form, n=_log(rng, 8, 20000 if form == "doppler" else 60000),
                        n_slots=_log(rng, 300, 4096), n_det=rng.randint(1, 3), K=rng.choice((4, 8, 8, 8, 13)))
        if data == "space":
            return dict(kind=kind, data=data, form="plain", n=_log(rng, 500, 200000), n_slots=rng.randint(20, 60),
                        n_det=1, K=rng.choice((32, 32, 24)))
        if data == "bns":
            return dict(kind=kind, data=data, form="plain", n=_log(rng, 20, 1000), n_slots=_log(rng, 800, 6384),
                        n_det=1, K=rng.choice((50, 32, 21)))
        return dict(kind=kind, data=data, form="plain", n=_log(rng, 100, 100000), n_slots=rng.randint(60, 256),
                    n_det=1, K=rng.choice((4, 4, 6)), waveform=rng.choice(("newton", "pn35")),
                    precision=rng.choice(("fp64", "fp32_kahan")))
    if kind == "sfts":
        if rng.random() < 0.5:
            n = 1 << rng.randint(8, 13)
            w = rng.choice((8, 16, 25, 32, 50))
            return dict(kind=kind, n_samples=n, n_seg=max(3, _log(rng, 100, 4 << 20) // n // (8 if w > 32 else 1)),
                        n_det=rng.randint(1, 3), w=w)
        n = 2 * rng.randint(300, 3000)
        return dict(kind=kind, n_samples=n, n_seg=max(3, _log(rng, 40000, 12 << 20) // n), n_det=1, w=0) if n & (n - 1) \
            else dict(kind=kind, n_samples=n + 2, n_seg=99, n_det=1, w=0)
    if kind == "infer":
        return dict(kind=kind, mode=rng.choice(("fp64", "fp64", "bf16x3", "bf16")), hidden=rng.choice((32, 64, 96, 128)),
                    layers=rng.randint(2, 4), n=_log(rng, 500, 1 << 20))
    if kind == "train":
        return dict(kind=kind, hidden=rng.choice((32, 64, 96, 128)), layers=rng.randint(2, 4),
                    batch=_log(rng, 500, 4096), steps=rng.randint(8, 32))
    return dict(kind=kind, mode=rng.choice(("fp64", "bf16x3", "bf16")), hidden=rng.choice((64, 128)),
                layers=rng.randint(2, 4), n=_log(rng, 100, 16000), n_slots=rng.randint(60, 256), K=4)


# ------------------------------------------------------------------------------------ inputs
class _Draws:
    """Random numbers on the device from a seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def normal(self, *shape):
        return torch.randn(shape, dtype=torch.float64, device=DEV, generator=self.g)

    def uniform(self, lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(shape, dtype=torch.float64, device=DEV, generator=self.g)

    def integers(self, lo, hi, *shape):   # lo .. hi inclusive
        return torch.randint(lo, hi + 1, shape, device=DEV, generator=self.g)


def _orbit(t, radius, period, phase, tilt):
    W = 2.0 * math.pi / period
    c, s = np.cos(W * t + phase), np.sin(W * t + phase)
    ct, st = math.cos(tilt), math.sin(tilt)
    r = radius * np.stack([c, s * ct, s * st], -1)
    v = radius * W * np.stack([-s, c * ct, c * st], -1)
    return np.concatenate([r, v, -(W * W) * r], -1)


def _dataset(case, rnd):
    """SFT rows of the case's data set: raw bins and PSD (device FP64), start times, patterns."""
    n_slots = case["n_slots"]
    name = case.get("data", "tiny" if case["kind"] == "sur" else "ground")
    if name == "ground":
        t_sft, fs, k_lo, k_hi = 32.0, 128.0, 32, 512
        n_keep = n_slots - int(round(0.05 * n_slots))
        slots = [torch.sort(torch.argsort(rnd.uniform(0, 1, n_slots))[:n_keep])[0].cpu().numpy() for _ in range(case["n_det"])]
        t = np.concatenate([s * t_sft for s in slots])
        det = np.repeat(np.arange(case["n_det"]), n_keep)
        f = torch.arange(k_lo, k_hi, dtype=torch.float64, device=DEV) / t_sft
        psd = rnd.uniform(0.8, 1.2, t.size)[:, None] * ((f / 5.0) ** -4 + 1.0 + (f / 50.0) ** 2)[None, :]
        ph = 2.0 * math.pi * (t + 0.5 * t_sft) / DAY + 2.0 * math.pi * det / 3.0
    elif name == "space":
        t_sft, fs, k_lo, k_hi = 2 * DAY, 0.2, 0, 1792
        t, det = np.arange(n_slots) * t_sft, np.zeros(n_slots, int)
        psd = torch.ones((n_slots, k_hi - k_lo), dtype=torch.float64, device=DEV)
        ph = 2.0 * math.pi * (t + 0.5 * t_sft) / YEAR
    else:
        t_sft, fs = (73.0, 40.0) if name == "bns" else (64.0, 32.0)
        k_lo, k_hi = 0, int(round(t_sft * fs)) // 2 + 1
        t, det = np.arange(n_slots) * t_sft, np.zeros(n_slots, int)
        psd = torch.full((n_slots, k_hi - k_lo), 1.0 if name == "bns" else 2.0 / fs, dtype=torch.float64, device=DEV)
        ph = None
    x = torch.complex(rnd.normal(*psd.shape), rnd.normal(*psd.shape)) * torch.sqrt(t_sft * psd / 4.0)
    d = dict(t=t, det=det, n=int(round(t_sft * fs)), T=t_sft, k_lo=k_lo, x=x, psd=psd,
             fp=None if ph is None else np.cos(ph), fx=None if ph is None else np.sin(ph), eph=None)
    if case.get("form") == "doppler":
        # Earth's orbit (in the ecliptic) and rotation at each detector's site
        e = np.empty((t.size, 9))
        for i, (lat, lon) in enumerate(SITES):
            m = det == i
            tm = t[m] + 0.5 * t_sft
            e[m] = _orbit(tm, 499.00478383615643, YEAR, 0.0, math.radians(23.4393))
            e[m] += _orbit(tm, 6.371e6 / 299792458.0 * math.cos(lat), 86164.0905, lon, 0.0)
            e[m, 2] += 6.371e6 / 299792458.0 * math.sin(lat)
        d["eph"] = e
    return d


def _bank(case, d, rnd):
    """The template bank (device tensors) in the order that a bank generator gives it: by mass."""
    n = case.get("n", 1)
    name = case.get("data", "tiny" if case["kind"] == "sur" else "ground")
    n_sft = d["t"].size
    if name == "space":
        mc = torch.exp(rnd.uniform(math.log(1e5), math.log(1e6), n))
        n_use = rnd.integers(min(8, n_sft), n_sft, n)
        o = torch.argsort(n_use.double() * -1e3 + torch.log(mc))   # by range, then by mass
        mc, n_use = mc[o], n_use[o]
        t_c = d["t"][-1] + 0.5 * d["T"] + 3.5e5 * (mc / 1e5) ** (-5.0 / 19.0)
        return dict(mc=mc, t_c=t_c, phi_c=torch.zeros_like(mc), a_first=(n_sft - n_use).to(torch.int32),
                    a_last=torch.full((n,), n_sft - 1, dtype=torch.int32, device=DEV))
    if name == "ground":
        lo, hi, t_c = 1.0, 1.5, case["n_slots"] * d["T"] + 600.0
    elif name == "bns":
        mc0 = 1.4 / 2.0 ** 0.2
        M = mc0 * TSUN
        lo, hi, t_c = 0.995 * mc0, 1.005 * mc0, n_sft * d["T"] + 5.0 * M * (8.0 * math.pi * M * 10.0) ** (-8.0 / 3.0)
    else:
        lo, hi, t_c = 1.19, 1.21, n_sft * d["T"] + 600.0
    mc = torch.sort(rnd.uniform(lo, hi, n))[0]
    b = dict(mc=mc, t_c=torch.full_like(mc, t_c), phi_c=rnd.uniform(0, 2 * math.pi, n))
    if case.get("waveform") == "pn35" or case["kind"] == "sur":
        b["q"] = rnd.uniform(1.0, 2.0, n)
    if case.get("form") == "doppler":
        ra, sd = rnd.uniform(0, 2 * math.pi, n), rnd.uniform(-1, 1, n)
        cd = torch.sqrt(1.0 - sd * sd)
        b["sky"] = torch.stack([cd * torch.cos(ra), cd * torch.sin(ra), sd], -1).contiguous()
    return b


def _options(case):
    tiny = case.get("data") == "tiny" or case["kind"] == "sur"
    o = dict(K=case["K"], kernel="dirichlet" if tiny else "auto", precision=case.get("precision", "fp32_kahan"),
             waveform=case.get("waveform", "newton"))
    if case.get("data", "ground") in ("ground", "space") and not tiny:
        o.update(a_plus=1.0, a_cross=1.0)
    return o


def _network(case, rnd):
    """Initial parameters W ~ N(0, 1 / n_in), output layer scaled by 0.1, biases small."""
    dims = [3] + [case["hidden"]] * case["layers"] + [2]
    parts = []
    for i in range(len(dims) - 1):
        W = rnd.normal(dims[i], dims[i + 1]) / math.sqrt(dims[i]) * (0.1 if i == len(dims) - 2 else 1.0)
        parts += [W.reshape(-1), 0.05 * rnd.normal(dims[i + 1])]
    return torch.cat(parts).float()


def _inputs(case, seed):
    """Everything that a pass reads, from the seed alone."""
    rnd = _Draws(seed)
    kind = case["kind"]
    if kind in ("ip", "bank", "sur"):
        d = _dataset(case, rnd)
        s = dict(d=d, bank=_bank(case, d, rnd))
        if kind == "sur":
            s["par"] = _network(case, rnd)
        return s
    if kind == "sfts":
        n, n_seg = case["n_samples"], case["n_seg"]
        return dict(x=rnd.normal(case["n_det"], n * n_seg + n // 3))   # a remainder shorter than a segment
    if kind == "infer":
        return dict(par=_network(case, rnd), u=rnd.uniform(-1, 1, case["n"], 3))
    n = case["batch"] * case["steps"] + case["batch"] // 2
    u = rnd.uniform(-1, 1, n, 3).float()
    y = torch.stack([0.6 * torch.sin(2.0 * u[:, 2] + u[:, 0]) + 0.2 * u[:, 1], 0.5 * u[:, 2] ** 2 - 0.3 * u[:, 0]], -1)
    return dict(par=_network(case, rnd), u=u, y=y.contiguous())


def _band(case):
    """Band of an SFT case: 15 of 64 bins from n/128 for estimated noise, every bin for a white level."""
    n = case["n_samples"]
    return (max(1, n // 128), max(8, 15 * n // 128)) if case["w"] else (0, n // 2 + 1)


# --------------------------------------------------------------------------- prepare and run
def prepare(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    st = dict(case=case)
    if kind in ("ip", "bank", "sur"):
        d = s["d"]
        storage = "f64" if case.get("precision") == "fp64" else "f32"
        st["data"] = sft.SFTData(d["t"], d["n"], d["T"], d["k_lo"], d["x"].cpu().numpy(), d["psd"].cpu().numpy(),
                                 d["fp"], d["fx"], storage=storage)
        if d["eph"] is not None:
            st["data"].set_ephemeris(d["eph"])
        o = _options(case)
        if kind == "sur":
            st["net"] = sft.Surrogate(s["par"].cpu().numpy(), hidden=case["hidden"], layers=case["layers"], head=1,
                                      judge_tol=1.0, inference=case["mode"], **SUR)
            o.update(waveform="surrogate", surrogate=st["net"])
        st["opts"] = sft.make_opts(**o)
        if kind == "ip":
            st["arg"] = {k: float(s["bank"][k][0]) for k in ("mc", "t_c", "phi_c")}
        else:
            st["bank"] = s["bank"]
            st["out"] = sft.alloc_out(case["n"], mismatch=kind == "sur", fstat=case.get("form") in ("fstat", "doppler"))
    elif kind == "sfts":
        st["x"] = s["x"]
    else:
        st["net"] = sft.Surrogate(s["par"].cpu().numpy(), hidden=case["hidden"], layers=case["layers"], head=1,
                                  inference=case.get("mode", "fp64"), **SUR)
        st["u"], st["y"] = s["u"], s.get("y")
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "ip":
        r = sft.inner_product(st["data"], opts=st["opts"], **st["arg"])
        r["zp"], r["zx"] = [r["zp"].real, r["zp"].imag], [r["zx"].real, r["zx"].imag]
        return r
    if kind in ("bank", "sur"):
        return sft.template_bank_scan(st["data"], st["bank"], st["opts"], out=st["out"])
    if kind == "sfts":
        k_lo, n_bins = _band(case)
        dt = 1.0 / 128.0 if case["w"] else 1.0 / 40.0
        bins, psd, keep = sft.make_sfts(st["x"], case["n_samples"], dt, k_lo, n_bins, case["w"],
                                        s_white=0.0 if case["w"] else 2.0 * dt)
        return dict(bins=bins, psd=psd, keep=keep)
    if kind == "infer":
        y, dy = st["net"].infer(st["u"])
        return dict(y=y, dy=dy)
    loss = st["net"].train(st["u"][: case["batch"] * case["steps"]], st["y"][: case["batch"] * case["steps"]],
                           batch=case["batch"], epochs=1, lr=1e-3, lr_min=1e-5)
    return dict(loss=loss, params=st["net"].get_params())


# ------------------------------------------------------------------------------------- exact
def _newton(m, tau, T):
    M = m["mc"] * TSUN
    y = tau / (5.0 * M)
    s = y ** -0.125
    kappa = s ** 3 * T / (8.0 * math.pi * M)
    return dict(kappa=kappa, phase=m["phi_c"] - 2.0 * y * s ** 3, amp=0.25 * s * s, beta=0.375 * kappa * T / tau)


def _masses(m):
    nu = m["q"] / (1.0 + m["q"]) ** 2
    return nu, m["mc"] * nu ** -0.6 * TSUN


def _phase_head(nu, th):
    """1PN and 1.5PN part of the phase series and its derivative in Theta."""
    p2, p3 = 3715.0 / 8064.0 + 55.0 / 96.0 * nu, -0.75 * math.pi
    return (-2.0 / nu * (p2 * th ** 0.375 + p3 * th ** 0.25),
            -2.0 / nu * (0.375 * p2 * th ** -0.625 + 0.25 * p3 * th ** -0.75))


def _pn35(m, tau, T):
    """The 3.5PN inspiral (TaylorT3 series in Theta = nu tau / 5M; Blanchet, Living Rev. Relativ. 17, 2)."""
    nu, M = _masses(m)
    pi, eul = math.pi, 0.57721566490153286061
    th = nu * tau / (5.0 * M)
    L = torch.log(th)
    s = th ** -0.125
    L256 = L - math.log(256.0)
    p = [3715.0 / 8064.0 + 55.0 / 96.0 * nu, -0.75 * pi + 0 * nu,
         9275495.0 / 14450688.0 + 284875.0 / 258048.0 * nu + 1855.0 / 2048.0 * nu ** 2,
         (-38645.0 / 172032.0 + 65.0 / 2048.0 * nu) * pi * L,
         831032450749357.0 / 57682522275840.0 - 53.0 / 40.0 * pi ** 2 - 107.0 / 56.0 * eul + 107.0 / 448.0 * L256
         + (-126510089885.0 / 4161798144.0 + 2255.0 / 2048.0 * pi ** 2) * nu + 154565.0 / 1835008.0 * nu ** 2
         - 1179625.0 / 1769472.0 * nu ** 3,
         (188516689.0 / 173408256.0 + 488825.0 / 516096.0 * nu - 141769.0 / 516096.0 * nu ** 2) * pi]
    phase = m["phi_c"] - 2.0 / nu * th * s ** 3 * (1.0 + sum(c * s ** (k + 2) for k, c in enumerate(p)))
    one = torch.ones_like(th)
    g6 = -107.0 / 3360.0
    q = {0: one, 2: 743.0 / 4032.0 + 11.0 / 48.0 * nu, 3: -0.2 * pi * one,
         4: 19583.0 / 254016.0 + 24401.0 / 193536.0 * nu + 31.0 / 288.0 * nu ** 2,
         5: (-11891.0 / 53760.0 + 109.0 / 1920.0 * nu) * pi,
         6: -10052469856691.0 / 6008596070400.0 + pi ** 2 / 6.0 + 107.0 / 420.0 * eul + g6 * L256
         + (3147553127.0 / 780337152.0 - 451.0 / 3072.0 * pi ** 2) * nu - 15211.0 / 442368.0 * nu ** 2
         + 25565.0 / 1327104.0 * nu ** 3,
         7: (-113868647.0 / 433520640.0 - 31821.0 / 143360.0 * nu + 294941.0 / 3870720.0 * nu ** 2) * pi}
    x = 0.25 * sum(c * s ** (k + 2) for k, c in q.items())
    # d/dTheta of c Theta^-(k+2)/8, with dc/dTheta = g6 / Theta for k = 6
    dx = 0.25 * sum((-(k + 2) / 8.0 * c + (g6 if k == 6 else 0.0)) * s ** (k + 10) for k, c in q.items())
    f = x ** 1.5 / (pi * M)
    amp = nu ** 0.4 * x * (1.0 + x * (-107.0 / 42.0 + 55.0 / 42.0 * nu) + 2.0 * pi * x ** 1.5
                           + x * x * (-2173.0 / 1512.0 - 1069.0 / 216.0 * nu + 2047.0 / 1512.0 * nu ** 2))
    return dict(kappa=f * T, phase=phase, amp=amp, beta=-1.5 * torch.sqrt(x) * dx * nu / (5.0 * M) / (pi * M) * T * T)


def _forward(par, hidden, layers, u):
    """Network and its derivative along the third input, FP64."""
    dims = [3] + [hidden] * layers + [2]
    h, t = u, torch.tensor([0.0, 0.0, 1.0], dtype=torch.float64, device=DEV).expand(u.shape[0], 3)
    at = 0
    for i in range(len(dims) - 1):
        W = par[at: at + dims[i] * dims[i + 1]].reshape(dims[i], dims[i + 1])
        at += W.numel()
        b = par[at: at + dims[i + 1]]
        at += dims[i + 1]
        h, t = h @ W + b, t @ W
        if i < layers:
            g = torch.sigmoid(h)
            h, t = h * g, g * (1.0 + h * (1.0 - g)) * t
    return h, t


def _surrogate(m, tau, T, par, case):
    """The surrogate chirp: the leading-order chirp, the analytic phase head and the network."""
    lo, hi = SUR["ln_tau"]
    u = torch.stack([2.0 * (m["mc"] - 1.19) / (1.21 - 1.19) - 1.0, 2.0 * (m["q"] - 1.0) - 1.0,
                     2.0 * (torch.log(tau) - lo) / (hi - lo) - 1.0], -1)
    y, dy = _forward(par.double(), case["hidden"], case["layers"], u)
    c = _newton(m, tau, T)
    Phi = (tau / (5.0 * m["mc"] * TSUN)) ** 0.125
    nu, M = _masses(m)
    hp, hd = _phase_head(nu, nu * tau / (5.0 * M))
    dphi = hp + SUR["c_phi"] * Phi * y[:, 0]
    ddphi = hd * nu / (5.0 * M) + SUR["c_phi"] * Phi * (0.125 * y[:, 0] + dy[:, 0] * 2.0 / (hi - lo)) / tau
    kappa = c["kappa"] - ddphi * T / (2.0 * math.pi)
    return dict(kappa=kappa, phase=c["phase"] + dphi, amp=c["amp"] * torch.exp(SUR["c_amp"] * y[:, 1]),
                beta=c["beta"] * (kappa / c["kappa"]) ** (11.0 / 3.0))


def _exact_scan(case, s):
    """The inner products by their definition: every kernel weight int exp(i (2 pi x s + pi beta s^2)) ds
    by Gauss-Legendre quadrature over the SFT, sums over the window and over the rows in FP64."""
    d, bank, o = s["d"], s["bank"], _options(case)
    K, T, n = o["K"], d["T"], bank["mc"].numel()
    xb = torch.where(d["psd"] > 0, torch.conj(2.0 * d["x"] / d["psd"]), torch.zeros_like(d["x"]))
    nyq, k_ext = d["n"] // 2, d["k_lo"]
    if d["k_lo"] == 0:                                  # mirrors of DC and of the Nyquist bin
        k_ext = -64
        xb = torch.cat([torch.conj(torch.flip(xb[:, 1:65], [1])), xb], 1)
    if d["k_lo"] + d["psd"].shape[1] - 1 == nyq:
        xb = torch.cat([xb, torch.conj(torch.flip(xb[:, -65:-1], [1]))], 1)
    n_ext, n_bins = xb.shape[1], d["psd"].shape[1]
    xb, psd = xb.reshape(-1), d["psd"].reshape(-1)
    # rows of one start time share the waveform, unless the detectors move
    doppler = "sky" in bank
    if doppler:
        order = np.argsort(d["t"], kind="stable")
        tm, rows = d["t"][order] + 0.5 * T, order[:, None]
    else:
        ut, inv = np.unique(d["t"], return_inverse=True)
        tm, rows = ut + 0.5 * T, np.full((ut.size, int(d["det"].max()) + 1), -1)
        rows[inv, d["det"]] = np.arange(d["t"].size)
    dev = lambda a, t=torch.float64: torch.as_tensor(np.ascontiguousarray(a), dtype=t, device=DEV)
    tm, rows = dev(tm), dev(rows, torch.int64)
    fp = dev(np.ones(d["t"].size) if d["fp"] is None else d["fp"])
    fx = dev(np.zeros(d["t"].size) if d["fx"] is None else d["fx"])
    eph = dev(d["eph"]) if doppler else None
    fresnel = o["kernel"] != "dirichlet"
    Q = 48 if not fresnel or K <= 16 and case.get("data", "ground") == "ground" else 224
    nodes, gw = np.polynomial.legendre.leggauss(Q)
    sq, gw = dev(0.5 * nodes), dev(0.5 * gw)
    j = torch.arange(-K, K + 1, dtype=torch.float64, device=DEV)
    E = torch.polar(gw[:, None].expand(Q, 2 * K + 1).contiguous(), -2.0 * math.pi * sq[:, None] * j[None, :])
    E = E * (1.0 - 2.0 * (torch.abs(j) % 2))            # (-1)^j
    ji = torch.arange(-K, K + 1, device=DEV)
    acc = torch.zeros((8, n), dtype=torch.float64, device=DEV)   # z+ (2), zx (2), hh+, hhx, hh+x
    jud = torch.zeros((3, n), dtype=torch.float64, device=DEV)
    af, al = bank.get("a_first"), bank.get("a_last")
    P = max(1, (1 << 23) // Q)
    nc = min(n, P)
    gb = max(1, P // nc)
    for m0 in range(0, n, nc):
        bm = {k: v[m0: m0 + nc] for k, v in bank.items()}
        nn = bm["mc"].numel()
        for g0 in range(0, tm.numel(), gb):
            ng = min(gb, tm.numel() - g0)
            m = {k: v.repeat(ng, *([1] * (v.dim() - 1))) for k, v in bm.items()}
            t = tm[g0: g0 + ng].repeat_interleave(nn)
            r = rows[g0: g0 + ng].repeat_interleave(nn, 0)
            if doppler:
                e = eph[r[:, 0]]
                dl, dv, da = ((e[:, 3 * i: 3 * i + 3] * m["sky"]).sum(1) for i in range(3))
                t = t + dl
            tau = m["t_c"] - t
            ok = tau > 0
            tau = torch.where(ok, tau, torch.ones_like(tau))
            if case["kind"] == "sur":
                c = _surrogate(m, tau, T, s["par"], case)
            else:
                c = (_pn35 if o["waveform"] == "pn35" else _newton)(m, tau, T)
            if doppler:
                c["beta"] = c["beta"] * (1.0 + dv) ** 2 + c["kappa"] * da * T
                c["kappa"] = c["kappa"] * (1.0 + dv)
            k0 = torch.floor(c["kappa"] + 0.5)
            ok &= (k0 >= 0) & (k0 <= nyq)
            k0 = torch.where(ok, k0, torch.zeros_like(k0))
            delta = torch.where(ok, c["kappa"] - k0, torch.zeros_like(k0))
            beta = torch.where(ok, c["beta"], torch.zeros_like(k0)) if fresnel else torch.zeros_like(k0)
            ph = 2.0 * math.pi * delta[:, None] * sq + math.pi * beta[:, None] * (sq * sq)
            w = torch.polar(torch.ones_like(ph), ph) @ E
            z = torch.polar(c["amp"] * (1.0 - 2.0 * (k0 % 2)), torch.remainder(c["phase"], 2.0 * math.pi))
            idx = k0.long()[:, None] + ji - k_ext
            inb = (idx >= 0) & (idx < n_ext)
            w = torch.where(inb, w, torch.zeros_like(w))
            idx = idx.clamp(0, n_ext - 1)
            kf = torch.floor(c["kappa"])
            ip = torch.where(ok, kf, torch.zeros_like(kf)).long() - d["k_lo"]
            pin = ok & (ip >= 0) & (ip + 1 < n_bins)
            ip = ip.clamp(0, n_bins - 2)
            lam = c["kappa"] - kf
            for k in range(r.shape[1]):
                rk = r[:, k]
                act = ok & (rk >= 0)
                if af is not None:
                    act &= (rk >= m["a_first"]) & (rk <= m["a_last"])
                rk = rk.clamp(min=0)
                C = (w * xb[rk[:, None] * n_ext + idx]).sum(1) * z
                C = torch.where(act, C, torch.zeros_like(C))
                S = (1.0 - lam) * psd[rk * n_bins + ip] + lam * psd[rk * n_bins + ip + 1]
                h = torch.where(act & pin, c["amp"] ** 2 * T / S, torch.zeros_like(S))
                a, b = fp[rk], fx[rk]
                terms = torch.stack([a * C.real, a * C.imag, b * C.real, b * C.imag, a * a * h, b * b * h, a * b * h])
                acc[:7, m0: m0 + nn] += terms.reshape(7, ng, nn).sum(1)
                if case["kind"] == "sur":
                    pn = _pn35(m, tau, T)
                    kp = torch.floor(pn["kappa"])
                    i0 = kp.long() - d["k_lo"]
                    pi = act & (i0 >= 0) & (i0 + 1 < n_bins)
                    i0 = i0.clamp(0, n_bins - 2)
                    lp = pn["kappa"] - kp
                    Sp = (1.0 - lp) * psd[rk * n_bins + i0] + lp * psd[rk * n_bins + i0 + 1]
                    wt = torch.where(pi, pn["amp"] ** 2 * T / Sp, torch.zeros_like(Sp))
                    dp, sc = c["phase"] - pn["phase"], torch.sinc(c["kappa"] - pn["kappa"])
                    js = torch.stack([wt * torch.cos(dp) * sc, wt * torch.sin(dp) * sc, wt])
                    jud[:, m0: m0 + nn] += js.reshape(3, ng, nn).sum(1)
    ap, ax = o.get("a_plus", 1.0), o.get("a_cross", 0.0)
    re, im = ap * acc[0] + ax * acc[3], ap * acc[1] - ax * acc[2]
    hh = ap * ap * acc[4] + ax * ax * acc[5]
    rho = torch.where(hh > 0, torch.sqrt(re * re + im * im) / torch.sqrt(hh), torch.zeros_like(hh))
    out = dict(zp=acc[0:2].t().contiguous(), zx=acc[2:4].t().contiguous(), hhp=acc[4], hhx=acc[5], rho=rho,
               flags=None, n_used=None)
    if case.get("form") in ("fstat", "doppler"):
        A, B, C, D = acc[4], acc[5], acc[6], acc[4] * acc[5] - acc[6] ** 2
        full = (B * (acc[0] ** 2 + acc[1] ** 2) + A * (acc[2] ** 2 + acc[3] ** 2)
                - 2.0 * C * (acc[0] * acc[2] + acc[1] * acc[3])) / D
        lmax = 0.5 * (A + B) + torch.hypot(0.5 * (A - B), C)
        u0, u1 = torch.where(A >= B, lmax - B, C), torch.where(A >= B, C, lmax - A)
        un = torch.hypot(u0, u1)
        part = (((u0 * acc[0] + u1 * acc[2]) / un) ** 2 + ((u0 * acc[1] + u1 * acc[3]) / un) ** 2) / lmax
        out.update(hhpx=C, twoF=torch.where((D >= 1e-2 * A * B) & (D > 0), full, part))
    if case["kind"] == "sur":
        out["mismatch"] = 1.0 - torch.sqrt(jud[0] ** 2 + jud[1] ** 2) / jud[2]
    return out


def _exact_sfts(case, x):
    n, n_seg, w = case["n_samples"], case["n_seg"], case["w"]
    k_lo, n_bins = _band(case)
    dt = 1.0 / 128.0 if w else 1.0 / 40.0
    bins = torch.empty((case["n_det"], n_seg, n_bins), dtype=torch.complex128, device=DEV)
    psd = torch.full((case["n_det"], n_seg, n_bins), 2.0 * dt, dtype=torch.float64, device=DEV)
    M = n // 2
    k = torch.arange(k_lo, k_lo + n_bins, device=DEV)
    blk = (k - w).clamp(0, M - 2 * w)[:, None] + torch.arange(2 * w + 1, device=DEV)
    B = sum(1.0 / (2 * w + 1 - i) for i in range(w + 1))
    step = max(1, (1 << 25) // (n_bins * (2 * w + 1) + n))
    for a in range(case["n_det"]):
        seg = x[a, : n * n_seg].reshape(n_seg, n)
        for i in range(0, n_seg, step):
            X = torch.fft.rfft(seg[i: i + step]) * dt
            bins[a, i: i + step] = X[:, k]
            if w:
                med = torch.sort((X.real ** 2 + X.imag ** 2)[:, blk], -1)[0][..., w]
                psd[a, i: i + step] = med * 2.0 / (n * dt * B)
    return dict(bins=bins, psd=psd, keep=None)


def _shuffled(n, steps_done):
    """The order in which an epoch visits its n rows: a keyed bijection (see sft_surrogate_train)."""
    h = 1
    while (1 << (2 * h)) < n:
        h += 1
    key = np.uint32(0x243F6A88 ^ ((steps_done * 0x85A308D3) & 0xFFFFFFFF))
    mask = np.uint32((1 << h) - 1)

    def once(x):
        L, R = x >> np.uint32(h), x & mask
        for r in range(4):
            v = R ^ np.uint32((int(key) + 0x9E3779B9 * (r + 1)) & 0xFFFFFFFF)
            for shift, mul in ((16, 0x7FEB352D), (15, 0x846CA68B)):
                v = (v ^ (v >> np.uint32(shift))) * np.uint32(mul)
            v = v ^ (v >> np.uint32(16))
            L, R = R, L ^ (v & mask)
        return (L << np.uint32(h)) | R
    x = once(np.arange(n, dtype=np.uint32))
    while (x >= n).any():
        x = np.where(x >= n, once(x), x)
    return torch.as_tensor(x.astype(np.int64), device=DEV)


def _exact_train(case, s):
    """The same 32 or fewer Adam steps in FP64."""
    n, B = case["batch"] * case["steps"], case["batch"]
    p = s["par"].double().requires_grad_(True)
    m1, m2 = torch.zeros_like(p), torch.zeros_like(p)
    order = _shuffled(n, 0)
    u, y = s["u"][:n].double()[order], s["y"][:n].double()[order]
    dims = [3] + [case["hidden"]] * case["layers"] + [2]
    total = 0.0
    for it in range(case["steps"]):
        h, at = u[it * B: (it + 1) * B], 0
        for i in range(len(dims) - 1):
            W = p[at: at + dims[i] * dims[i + 1]].reshape(dims[i], dims[i + 1])
            at += dims[i] * dims[i + 1]
            h = h @ W + p[at: at + dims[i + 1]]
            at += dims[i + 1]
            if i < case["layers"]:
                h = h * torch.sigmoid(h)
        loss = ((h - y[it * B: (it + 1) * B]) ** 2).sum() / B
        (g,) = torch.autograd.grad(loss, p)
        total += float(loss)
        lr = 1e-5 + 0.5 * (1e-3 - 1e-5) * (1.0 + math.cos(math.pi * it / case["steps"]))
        with torch.no_grad():
            m1.mul_(0.9).add_(g, alpha=0.1)
            m2.mul_(0.999).addcmul_(g, g, value=0.001)
            p -= lr * (m1 / (1.0 - 0.9 ** (it + 1))) / (torch.sqrt(m2 / (1.0 - 0.999 ** (it + 1))) + 1e-8)
    return dict(loss=torch.tensor([total / case["steps"]], dtype=torch.float64), params=p.detach())


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind in ("bank", "sur"):
        return _exact_scan(case, s)
    if kind == "ip":
        r = _exact_scan(dict(case, n=1), s)
        return dict(zp=[float(v) for v in r["zp"][0]], zx=[float(v) for v in r["zx"][0]], hhp=float(r["hhp"][0]),
                    hhx=float(r["hhx"][0]), rho=float(r["rho"][0]), flags=None)
    if kind == "sfts":
        return _exact_sfts(case, s["x"])
    if kind == "infer":
        y, dy = _forward(s["par"].double(), case["hidden"], case["layers"], s["u"])
        return dict(y=y, dy=dy)
    return _exact_train(case, s)


# -------------------------------------------------------------------------------------- work
def _scan_flops(n, groups, rows, K, fresnel):
    """Per (template, timestamp): chirp, phases and norm (about 300); per window bin: the kernel
    weight (2 endpoint terms, about 40, or one division) and a complex multiply-add per row."""
    return n * groups * (300.0 + (2 * K + 1) * ((40.0 if fresnel else 4.0) + 8.0 * rows))


def work(case):
    kind = case["kind"]
    if kind in ("ip", "bank", "sur"):
        n, G = case.get("n", 1), case["n_slots"]
        name = case.get("data", "tiny" if kind == "sur" else "ground")
        nb = {"ground": 480, "space": 1792, "bns": 1461, "tiny": 1025}[name]
        sz = 2 if case.get("precision") == "fp64" else 1
        n_det = case.get("n_det", 1)
        rows = int(0.95 * G) * n_det if name == "ground" else G
        use = G * (0.55 if name == "space" else 0.95)
        bts = n * 100.0
        # every stored bin that some template's window covers, once (one template: its windows)
        bts += rows * min(nb, (2 * case["K"] + 1) * n) * 12.0 * sz
        if case.get("form") == "doppler":
            fl = _scan_flops(n, use * n_det, 1, case["K"], True) + n * use * n_det * 60.0
        else:
            fl = _scan_flops(n, use, n_det, case["K"], name != "tiny")
        if case.get("waveform") == "pn35":
            fl += n * use * 200.0
        if kind == "sur":
            H, L = case["hidden"], case["layers"]
            fl += n * G * (4.0 * (3 * H + (L - 1) * H * H + 2 * H) + 600.0)
        return dict(bytes=bts, flops=fl)
    if kind == "sfts":
        n, segs = case["n_samples"], case["n_seg"] * case["n_det"]
        return dict(bytes=segs * (8.0 * n + 24.0 * _band(case)[1]), flops=segs * 2.5 * n * math.log2(n))
    H, L = case["hidden"], case["layers"]
    P = 3 * H + (L - 1) * H * H + 2 * H
    if kind == "infer":
        return dict(bytes=case["n"] * 56.0 + P * 8.0, flops=case["n"] * 4.0 * P)
    rows = case["batch"] * case["steps"]
    return dict(bytes=rows * 20.0 + case["steps"] * P * 28.0, flops=rows * 6.0 * P)
