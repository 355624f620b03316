"""Workloads that stand for the use of this map-making library, for timing it.

Every case is a survey (scan geometry, stationary intervals, noise model) and one call that a
map-making program makes on it: whole solves, Monte Carlo batches, single operators on ragged
data, a gradient step.  The geometries are those of the synthetic scans of this repository
(cross-linked IQU rasters, intensity rasters, ring scans, batches of rotated rasters), written
here with torch so that the inputs are made on the GPU.
"""

import math

import numpy as np
import torch

from paper_1408_3048_amd import Plan
from paper_1408_3048_amd.autograd import gls_map

F_SAMP = 200.0
HWP_HZ = 2.0
DET_DEG = (0.0, 45.0, 90.0, 135.0)
DEV = "cuda"

# PCG steps of one pass, rounded: what a solve of the kind takes on its surveys
STEPS = {"tts": 70, "batch": 30, "zd": 420, "small": 55, "solve64": 70, "grad": 160, "adjoint": 125}


def listed():
    return [
        # The smallest calls: one operator application on a 16x16 patch, where launches count
        # (an outer solver of the user's own, a test problem).
        dict(name="A-fp64-2e14", kind="A64", side=16, spp=8, cut=512, ragged=False, lam=64),
        # A training step through the autograd function on the 16x16 patch: the map of a TOD, a
        # loss of the map, gradients for the TOD and every interval's noise parameters.
        dict(name="grad-step-2e14", kind="grad", side=16, spp=8, cut=512, ragged=False, lam=64),
        # A new right-hand side on the kept plan of the intensity raster (2^18 samples, 16
        # passes): FP64 block Jacobi.
        dict(name="solve-I-2e18", kind="small", side=64, spp=4, passes=16, cut=1 << 14,
             ragged=False, lam=1024),
        # The FP64 operator on a survey as it comes: odd patch, no two intervals alike.
        dict(name="A-fp64-ragged", kind="A64", side=181, spp=8, cut=30011, ragged=True, lam=1500),
        # A first look at new data: plan, right-hand side and block-Jacobi map from an FP32 TOD
        # cut at arbitrary samples.
        dict(name="first-look-ragged", kind="look", side=250, spp=7, cut=40009, ragged=True,
             lam=2048),
        # The forward chain of a Monte Carlo run in FP32: simulate the TOD of a sky, add noise,
        # weight, bin.
        dict(name="simulate-weight-bin", kind="tod32", side=300, spp=8, cut=16411, ragged=True,
             lam=512),
        # Strong 1/f noise: the a posteriori coarse space from the first data set, then the
        # next data set solved with it.
        dict(name="krylov-space-2e20", kind="zd", side=128, spp=8, cut=1 << 15, ragged=False,
             lam=2048),
        # FP64 two-level solve of a new right-hand side on the 2^22-sample raster.
        dict(name="solve-fp64-2lvl-2e22", kind="solve64", side=256, spp=8, cut=1 << 17,
             ragged=False, lam=2048),
        # Gradients of a loss of the map on the 2^22-sample raster, map and plan in hand.
        dict(name="adjoint-2e22", kind="adjoint", side=256, spp=8, cut=1 << 17, ragged=False,
             lam=2048),
        # A batch of independent problems of uneven length in one kept plan.
        dict(name="batch-48", kind="batch", problems=48, side=128, n_min=1 << 16, n_max=1 << 20,
             cut=1 << 14, lam=1024),
        # One GPU's share of the ring scan (two detectors): the mixed operator, pixels seen at
        # scattered times, wide band.
        dict(name="A-mixed-ring-2e25", kind="ring", per_det=1 << 24, lon=2048, lat=1024,
             cut=1 << 18, lam=4096),
        # Time to solution on the 2^24-sample raster: plan with its coarse space, right-hand
        # side, mixed two-level PCG.
        dict(name="map-mixed-2lvl-2e24", kind="tts", side=512, spp=8, cut=1 << 16, ragged=False,
             lam=2048),
    ]


def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    """One more case: a kind, a size over its range (by its logarithm), an interval length and
    band that go with it."""
    kind = rng.choice(["A64", "A64", "grad", "small", "look", "tod32", "zd", "solve64", "adjoint",
                       "batch", "ring", "tts"])
    if kind == "batch":
        n_max = _log(rng, 1 << 17, 1 << 20)
        return dict(kind=kind, problems=_log(rng, 3, 48), side=rng.randint(40, 128),
                    n_min=1 << 16, n_max=n_max, cut=_log(rng, 1 << 13, 1 << 15),
                    lam=rng.choice([512, 777, 1024]))
    if kind == "ring":
        return dict(kind=kind, per_det=_log(rng, 1 << 20, 1 << 24), lon=2048, lat=1024,
                    cut=_log(rng, 1 << 16, 1 << 18), lam=rng.choice([2048, 3001, 4096]))
    side = {"A64": (16, 400), "grad": (16, 48), "small": (32, 160), "look": (60, 400),
            "tod32": (60, 512), "zd": (48, 128), "solve64": (64, 256), "adjoint": (64, 256),
            "tts": (100, 512)}[kind]
    side = _log(rng, *side)
    case = dict(kind=kind, side=side, spp=rng.choice([5, 7, 8]))
    per_det = 2 * side * side * case["spp"]
    if kind == "small":
        case.update(spp=4, passes=rng.randint(5, 16))
        per_det = side * side * 4 * case["passes"]
    if kind == "grad":
        lam = rng.choice([64, 100, 128])
        cut = rng.randint(512, 2048)
    elif kind == "zd":
        lam = rng.choice([1024, 2048])
        cut = rng.randint(4 * lam, max(4 * lam, per_det // 4))
    else:
        lam = rng.choice([v for v in (64, 300, 512, 1024, 1500, 2048) if 16 * v <= per_det] or [64])
        cut = rng.randint(6 * lam, max(6 * lam, min(per_det, 1 << 17)))
    case.update(cut=cut, ragged=rng.random() < 0.5, lam=lam)
    return case


# ---------------------------------------------------------------- surveys


def _pass(side, spp, vertical):
    """Pixels of one boustrophedon pass over a side x side patch, spp samples per pixel."""
    k = torch.arange(side * side * spp, device=DEV)
    line, u = k // (side * spp), (k % (side * spp)) // spp
    along = torch.where(line % 2 == 1, side - 1 - u, u)
    row, col = (along, line) if vertical else (line, along)
    return (row * side + col).to(torch.int32)


def _cuts(n_det, per_det, cut, ragged):
    """Interval bounds: each detector's timeline in pieces of `cut` samples (the last one what is
    left), or of uneven lengths around it."""
    r = np.random.RandomState(12345)
    lens = []
    for _ in range(n_det):
        left = per_det
        while left > 0:
            n = int(cut * r.uniform(0.6, 1.4)) if ragged else cut
            n = left if left - n < cut // 2 else n
            lens.append(n)
            left -= n
    return np.concatenate([[0], np.cumsum(np.array(lens, dtype=np.int64))])


def _angles(t, det_deg):
    phi = math.radians(det_deg) + 4.0 * math.pi * HWP_HZ * t
    return torch.stack([torch.cos(2.0 * phi), torch.sin(2.0 * phi)], -1)


def _raster(case):
    side, spp = case["side"], case["spp"]
    if case["kind"] == "small":  # intensity only, one detector, identical passes
        pix = _pass(side, spp, False).repeat(case["passes"])
        off = _cuts(1, pix.numel(), case["cut"], case["ragged"])
        return dict(pix=pix, w=None, n_pix=side * side, off=off, ns=1, prob=None)
    one = torch.cat([_pass(side, spp, False), _pass(side, spp, True)])
    t = torch.arange(one.numel(), dtype=torch.float64, device=DEV) / F_SAMP
    w = torch.cat([_angles(t, d) for d in DET_DEG])
    off = _cuts(4, one.numel(), case["cut"], case["ragged"])
    return dict(pix=one.repeat(4), w=w, n_pix=side * side, off=off, ns=3, prob=None)


def _ring(case):
    """Two detectors of the spinning, slowly precessing great-circle scan."""
    n, n_lon, n_lat = case["per_det"], case["lon"], case["lat"]
    t = torch.arange(n, dtype=torch.float64, device=DEV) / F_SAMP
    a = math.radians(0.1) / 60.0 * t
    pix, w = [], []
    for d in range(2):
        cross, along = math.radians((d - 1.5) * 0.5), math.radians(-0.75)
        ph = 2.0 * math.pi / 60.0 * t + along
        ca, sa, cp, sp = torch.cos(a), torch.sin(a), torch.cos(ph), torch.sin(ph)
        cc, sc = math.cos(cross), math.sin(cross)
        bx, by, bz = cc * sp * sa + sc * ca, -cc * sp * ca + sc * sa, cc * cp
        colat = torch.acos(bz.clamp(-1.0, 1.0))
        lon = torch.remainder(torch.atan2(by, bx), 2.0 * math.pi)
        ilat = (colat / math.pi * n_lat).long().clamp(max=n_lat - 1)
        ilon = (lon / (2.0 * math.pi) * n_lon).long().clamp(max=n_lon - 1)
        pix.append((ilat * n_lon + ilon).to(torch.int32))
        vx, vy, vz = cp * sa, -cp * ca, -sp
        east = -vx * torch.sin(lon) + vy * torch.cos(lon)
        north = (-torch.cos(colat) * (vx * torch.cos(lon) + vy * torch.sin(lon))
                 + torch.sin(colat) * vz)
        phi = math.radians(d * 11.25) + 4.0 * math.pi * HWP_HZ * t + torch.atan2(east, north)
        w.append(torch.stack([torch.cos(2.0 * phi), torch.sin(2.0 * phi)], -1))
    return dict(pix=torch.cat(pix), w=torch.cat(w), n_pix=n_lon * n_lat,
                off=_cuts(2, n, case["cut"], False), ns=3, prob=None)


def _turned(n, side, theta):
    """A boustrophedon raster of n samples turned by theta, covering the patch's outer circle."""
    half = side * math.sqrt(2.0) / 2.0
    lines = max(2, int(math.sqrt(n / 2.0)))
    per = -(-n // lines)
    k = torch.arange(n, device=DEV)
    line = k // per
    u = ((k % per).double() + 0.5) / per
    u = torch.where(line % 2 == 1, 1.0 - u, u)
    x, y = 2.0 * half * u - half, 2.0 * half * (line.double() + 0.5) / lines - half
    c, s = math.cos(theta), math.sin(theta)
    return c * x - s * y + side / 2.0, s * x + c * y + side / 2.0


def _batch(case):
    """Independent problems: turned rasters of uneven length, samples off the patch dropped."""
    r = np.random.RandomState(777)
    side, pix, w, off, prob, base = case["side"], [], [], [0], [0], 0
    for b in range(case["problems"]):
        n = int(math.exp(r.uniform(math.log(case["n_min"]), math.log(case["n_max"])))) // 4
        theta = r.uniform(0.0, math.pi)
        xh, yh = _turned(n // 2, side, theta)
        xv, yv = _turned(n - n // 2, side, theta + math.pi / 2.0)
        x, y = torch.cat([xh, xv]), torch.cat([yh, yv])
        keep = (x >= 0) & (x < side) & (y >= 0) & (y < side)
        p = (y[keep].long() * side + x[keep].long() + b * side * side).to(torch.int32)
        t = torch.nonzero(keep)[:, 0].double() / F_SAMP
        for d in DET_DEG:
            pix.append(p)
            w.append(_angles(t, d))
            off += [base + min(k + case["cut"], p.numel()) for k in range(0, p.numel(), case["cut"])]
            base += p.numel()
        prob.append(len(off) - 1)
    return dict(pix=torch.cat(pix), w=torch.cat(w), n_pix=side * side * case["problems"],
                off=np.array(off, dtype=np.int64), ns=3, prob=np.array(prob, dtype=np.int32))


def _survey(case, seed):
    """The survey of a case with the noise parameters, sky and noise of a seed."""
    s = {"batch": _batch, "ring": _ring}.get(case["kind"], _raster)(case)
    rng = np.random.RandomState(seed % (1 << 31))
    k = len(s["off"]) - 1
    fk, al = {"batch": ((0.3, 5.0), (1.0, 1.0)), "ring": ((0.7, 1.3), (1.0, 1.0)),
              "small": ((0.7, 1.3), (1.0, 1.0)), "zd": ((1.8, 2.2), (2.0, 2.0)),
              }.get(case["kind"], ((0.5, 2.0), (1.0, 2.0)))
    if case["kind"] not in ("batch", "ring", "small") and case["lam"] < 1024:
        # a narrow band holds a 1/f spectrum only where its knee lies above the band's width
        fk = (max(2.0, 200.0 / case["lam"]), max(4.0, 400.0 / case["lam"]))
    s["psd"] = np.stack([rng.uniform(0.8, 1.2, k), rng.uniform(*fk, k), rng.uniform(*al, k)], 1)
    g = torch.Generator(device=DEV).manual_seed(seed)
    s["gen"] = g
    s["lam"] = case["lam"]
    n = s["pix"].numel()
    s["noise"] = _noise(s, torch.randn(n, dtype=torch.float64, device=DEV, generator=g))
    sky = torch.randn((s["n_pix"], s["ns"]), dtype=torch.float64, device=DEV, generator=g)
    sky[:, 1:] *= 0.1
    s["sky"] = sky
    return s


def _groups(s):
    """(length, starts, interval indices) of the intervals of each length."""
    off = s["off"]
    lens = np.diff(off)
    return [(int(n), off[:-1][lens == n], np.nonzero(lens == n)[0]) for n in np.unique(lens)]


def _rows(n, starts):
    return torch.from_numpy(starts).to(DEV)[:, None] + torch.arange(n, device=DEV)


def _noise(s, white):
    """White noise coloured to each interval's 1/f spectrum, zero frequency removed."""
    out = torch.empty_like(white)
    for n, starts, idx in _groups(s):
        p = torch.from_numpy(s["psd"][idx]).to(DEV)
        f = torch.arange(n // 2 + 1, dtype=torch.float64, device=DEV) * (F_SAMP / n)
        f[0] = 1.0
        amp = p[:, :1] * torch.sqrt(1.0 + (p[:, 1:2] / f) ** p[:, 2:3])
        amp[:, 0] = 0.0
        at = _rows(n, starts)
        out[at] = torch.fft.irfft(torch.fft.rfft(white[at]) * amp, n=n)
    return out


def _plan(s, **kw):
    return Plan(s["pix"], s["w"], s["n_pix"], s["off"], s["psd"], n_stokes=s["ns"], lam=s["lam"],
                f_samp=F_SAMP, problem_intervals=s["prob"], **kw)


def _compact_sky(s):
    """The sky at the observed pixels, as the library numbers them."""
    return s["sky"][torch.unique(s["pix"].long())].reshape(-1).contiguous()


def _signal(s):
    """The sky seen by every sample."""
    v = s["sky"][s["pix"].long()]
    if s["ns"] == 1:
        return v[:, 0].contiguous()
    return v[:, 0] + s["w"][:, 0] * v[:, 1] + s["w"][:, 1] * v[:, 2]


def _second_noise(s):
    n = s["pix"].numel()
    return _noise(s, torch.randn(n, dtype=torch.float64, device=DEV, generator=s["gen"]))


def _map_like(s, n):
    return torch.randn(n, dtype=torch.float64, device=DEV, generator=s["gen"])


# ---------------------------------------------------------------- the calls


def prepare(case, seed):
    kind = case["kind"]
    s = _survey(case, seed)
    st = dict(kind=kind)
    if kind in ("A64", "ring"):
        st["x"] = _compact_sky(s)
        st["plan"] = _plan(s, precision="mixed", rcond_min=0.0) if kind == "ring" else _plan(s)
    elif kind == "grad":
        st.update(d=_signal(s) + s["noise"], psd=torch.from_numpy(s["psd"]).to(DEV),
                  pix=s["pix"], w=s["w"], n_pix=s["n_pix"], off=s["off"], lam=s["lam"],
                  target=_compact_sky(s))
    elif kind == "look":
        st.update(s=s, d=(_signal(s) + s["noise"]).float())
    elif kind == "tts":
        st.update(s=s, d=_signal(s) + s["noise"])
    elif kind == "tod32":
        st.update(plan=_plan(s, precision="mixed"), x=_compact_sky(s), noise=s["noise"].float())
    elif kind == "zd":
        plan = _plan(s, precision="mixed")
        sig = _signal(s)
        st.update(plan=plan, b1=plan.rhs(sig + s["noise"]), b2=plan.rhs(sig + _second_noise(s)))
    elif kind in ("small", "solve64", "batch"):
        st.update(plan=_plan(s, precision="mixed" if kind == "batch" else "fp64",
                             coarse=kind != "small"), d=_signal(s) + s["noise"])
    else:  # adjoint: the map of the data is in hand
        plan = _plan(s)
        d = _signal(s) + s["noise"]
        m, _ = plan.pcg_solve(plan.rhs(d), tol=1e-12, max_iter=3000, history=False)
        st.update(plan=plan, d=d, m=m, g=2.0 * (m - _compact_sky(s)) / m.numel())
    return st


def run(st):
    """One pass.  Maps of mixed-precision operators and solves are good to about 1e-7 and are
    kept in FP32, as a program stores them."""
    kind = st["kind"]
    if kind == "A64":
        return st["plan"].apply_A(st["x"])
    if kind == "ring":
        return st["plan"].apply_A(st["x"], precision="mixed").float()
    if kind == "grad":
        d = st["d"].detach().requires_grad_(True)
        psd = st["psd"].detach().requires_grad_(True)
        m = gls_map(d, psd, st["pix"], st["w"], st["n_pix"], st["off"], n_stokes=3, lam=st["lam"],
                    f_samp=F_SAMP, tol=1e-11)
        loss = ((m - st["target"]) ** 2).mean()
        gd, gp = torch.autograd.grad(loss, (d, psd))
        return m.detach(), gd, gp
    if kind == "look":
        plan = _plan(st["s"], precision="mixed")
        b = plan.rhs(st["d"])
        m = plan.precond_bj(b)
        hits = plan.hits()
        plan.close()
        return b, m, hits
    if kind == "tts":
        plan = _plan(st["s"], precision="mixed", coarse=True)
        x, _ = plan.pcg_solve(plan.rhs(st["d"]), precond="2lvl", precision="mixed", tol=1e-8,
                              history=False)
        plan.close()
        return x.float()
    if kind == "tod32":
        d = st["plan"].apply_P(st["x"], dtype=torch.float32).add_(st["noise"])
        z = st["plan"].apply_Ninv(d, precision="mixed")
        return d, z, st["plan"].apply_PT(z).float()
    if kind == "zd":
        x1, _ = st["plan"].coarse_from_krylov(st["b1"], tol=1e-8, max_iter=2000, history=False)
        x2, _ = st["plan"].pcg_solve(st["b2"], precond="2lvl", precision="mixed", tol=1e-8,
                                     max_iter=2000, history=False)
        return x1.float(), x2.float()
    if kind == "small":
        b = st["plan"].rhs(st["d"])
        return b, st["plan"].pcg_solve(b, tol=1e-11, max_iter=5000,
                                          history=False)[0]
    if kind == "solve64":
        b = st["plan"].rhs(st["d"])
        return b, st["plan"].pcg_solve(b, precond="2lvl", tol=1e-11, max_iter=5000,
                                          history=False)[0]
    if kind == "batch":
        x, _ = st["plan"].pcg_solve(st["plan"].rhs(st["d"]), precond="2lvl", precision="mixed",
                                    tol=1e-8, history=False)
        return x.float()
    gd, gp, mu, _ = st["plan"].adjoint(st["m"], st["g"], st["d"], tol=1e-12)
    return gd, gp, mu


def _sizes(case):
    """(samples, pixels, Stokes parameters), of a drawn raster as planned."""
    if case["kind"] == "small":
        return case["side"] ** 2 * case["spp"] * case["passes"], case["side"] ** 2, 1
    if case["kind"] == "batch":
        a, b = math.log(case["n_min"]), math.log(case["n_max"])
        mean = (math.exp(b) - math.exp(a)) / (b - a) if b > a else math.exp(a)
        return int(0.5 * mean * case["problems"]), case["side"] ** 2 * case["problems"], 3
    if case["kind"] == "ring":  # the axis precesses by 0.1 deg a minute, both ends sweep the sky
        part = min(1.0, 2.0 * case["per_det"] / F_SAMP / 60.0 * 0.1 / 360.0)
        return 2 * case["per_det"], int(part * case["lon"] * case["lat"]) + 1, 3
    return 8 * case["side"] ** 2 * case["spp"], case["side"] ** 2, 3


def work(case):
    """Bytes and operations of one pass: the pointing (a pixel index and two weights for IQU)
    read once per application of A, maps read and written once; the band convolution as FFTs of
    twice the band's width."""
    n, p, ns = _sizes(case)
    kind = case["kind"]
    word = 4 if kind in ("ring", "tts", "tod32", "batch") else 8
    point = 4 + (2 * word if ns == 3 else 0)
    a_bytes = n * point + 2 * 8 * p * ns
    a_flops = n * (10.0 * math.log2(4.0 * case["lam"] + 4.0) + 4.0 * ns)
    times = STEPS.get(kind, 1)
    extra = 0
    if kind == "look":      # pointing and TOD in, the plan's sorted copy of the pointing out
        extra = n * (4 + 4 + 16) + n * (4 + 16)
    elif kind == "tts":     # the same, and the TOD of the right-hand side
        extra = n * (4 + 8 + 16) + n * (4 + 16)
    elif kind == "tod32":   # d and z out, noise in, pointing for P and P^T
        extra = n * (4 * 3 + point)
    elif kind == "grad":
        extra = n * (4 + 16 + 3 * 8)
    elif kind == "adjoint":  # d in, its gradient out, the lag correlations of two TODs
        extra = n * 4 * 8
    elif kind in ("small", "solve64", "batch"):
        extra = n * 8
    return dict(bytes=float(times * a_bytes + extra), flops=float(times * a_flops))


# ---------------------------------------------------------------- in 64 bits


class _Exact:
    """The operators of a survey in plain torch FP64: Toeplitz blocks by zero-padded FFTs of
    whole intervals, sums by index_add."""

    def __init__(self, s):
        self.s, self.ns = s, s["ns"]
        ids = s["pix"].long()
        obs = torch.unique(ids)
        self.cid = torch.searchsorted(obs, ids)
        self.n_obs = obs.numel()
        self.groups = []
        for n, starts, idx in _groups(s):
            m = 1 << (2 * n - 1).bit_length()
            t = self.taps(n, idx)
            row = torch.zeros((len(idx), m), dtype=torch.float64, device=DEV)
            row[:, :t.shape[1]] = t
            if t.shape[1] > 1:
                row[:, m - t.shape[1] + 1:] = t[:, 1:].flip(1)
            self.groups.append((n, m, _rows(n, starts), torch.fft.rfft(row).real, t, idx))

    def q(self, n, idx, what=0):
        p = torch.from_numpy(self.s["psd"][idx]).to(DEV)
        sg, fk, al = p[:, :1], p[:, 1:2], p[:, 2:3]
        f = torch.arange(n // 2 + 1, dtype=torch.float64, device=DEV) * (F_SAMP / n)
        f[0] = 1.0
        r = (fk / f) ** al
        q = 1.0 / (sg * sg * (1.0 + r))
        q = [q, -2.0 * q / sg, -q * (al * r / fk) / (1.0 + r),
             -q * r * torch.log(fk / f) / (1.0 + r)][what]
        q[:, 0] = 0.0
        return q

    def taps(self, n, idx, what=0):
        k = min(self.s["lam"], n - 1)
        x = torch.arange(k + 1, dtype=torch.float64, device=DEV) / self.s["lam"]
        return torch.fft.irfft(self.q(n, idx, what), n=n)[:, :k + 1] * torch.exp(-x * x)

    def ninv(self, y):
        z = torch.empty_like(y)
        for n, m, at, h, _, _ in self.groups:
            z[at] = torch.fft.irfft(torch.fft.rfft(y[at], n=m) * h, n=m)[:, :n]
        return z

    def P(self, x):
        v = x.reshape(-1, self.ns)[self.cid]
        w = self.s["w"]
        return v[:, 0] if self.ns == 1 else v[:, 0] + w[:, 0] * v[:, 1] + w[:, 1] * v[:, 2]

    def PT(self, z):
        w = self.s["w"]
        cols = [z] if self.ns == 1 else [z, w[:, 0] * z, w[:, 1] * z]
        out = torch.zeros((self.n_obs, self.ns), dtype=torch.float64, device=DEV)
        return out.index_add_(0, self.cid, torch.stack(cols, 1)).reshape(-1)

    def A(self, x):
        return self.PT(self.ninv(self.P(x)))

    def bj(self):
        t0 = torch.empty(self.s["pix"].numel(), dtype=torch.float64, device=DEV)
        for _, _, at, _, t, _ in self.groups:
            t0[at] = t[:, :1]
        w = self.s["w"]
        cols = [torch.ones_like(t0)] if self.ns == 1 else [torch.ones_like(t0), w[:, 0], w[:, 1]]
        blocks = torch.stack([self.PT(t0 * c).reshape(-1, self.ns) for c in cols], -1)
        inv = torch.linalg.inv(blocks)
        return lambda r: (inv @ r.reshape(-1, self.ns, 1)).reshape(-1)

    def solve(self, b, tol=1e-13, steps=1200):
        """A^-1 b by block-Jacobi CG, every problem of a batch under its own scalars."""
        prec, prob = self.bj(), self.s["prob"]
        of = torch.zeros(self.n_obs, dtype=torch.long, device=DEV)
        if prob is not None:
            first = torch.from_numpy(self.s["off"][prob[1:-1]]).to(DEV)
            of[self.cid] = torch.bucketize(torch.arange(self.cid.numel(), device=DEV), first,
                                           right=True)
        of = of.repeat_interleave(self.ns)
        k = 1 if prob is None else len(prob) - 1

        def dot(u, v):
            if k == 1:
                return (u * v).sum().reshape(1)
            return torch.zeros(k, dtype=torch.float64, device=DEV).index_add_(0, of, u * v)

        x, r = torch.zeros_like(b), b.clone()
        z = prec(r)
        p, rz, bb = z.clone(), dot(r, z), dot(b, b)
        for it in range(steps):
            q = self.A(p)
            a = (rz / dot(p, q).clamp(min=1e-300))[of]
            x, r = x + a * p, r - a * q
            if it % 10 == 9 and bool((dot(r, r) <= tol * tol * bb).all()):
                break
            z = prec(r)
            new = dot(r, z)
            p, rz = z + (new / rz.clamp(min=1e-300))[of] * p, new
        return x

    def gradients(self, d, m, mu):
        """dL/dd and dL/dpsd for mu = A^-1 dL/dm."""
        u, v = self.P(mu), d - self.P(m)
        gp = torch.zeros((len(self.s["off"]) - 1, 3), dtype=torch.float64, device=DEV)
        for n, m2, at, _, _, idx in self.groups:
            fu, fv = torch.fft.rfft(u[at], n=m2), torch.fft.rfft(v[at], n=m2)
            c = torch.fft.irfft(fu.conj() * fv + fu * fv.conj(), n=m2)
            for i in range(3):
                t = self.taps(n, idx, i + 1)
                cc = c[:, :t.shape[1]].clone()
                cc[:, 0] *= 0.5
                gp[torch.from_numpy(idx).to(DEV), i] = (t * cc).sum(1)
        return self.ninv(u), gp


def exact(case, seed):
    kind = case["kind"]
    s = _survey(case, seed)
    e = _Exact(s)
    if kind in ("A64", "ring"):
        return e.A(_compact_sky(s))
    if kind == "look":
        b = e.PT(e.ninv((_signal(s) + s["noise"]).float().double()))
        return b, e.bj()(b), None
    if kind == "tod32":
        d = e.P(_compact_sky(s)) + s["noise"].float().double()
        z = e.ninv(d)
        return d, z, e.PT(z)
    sig = _signal(s)
    d = sig + s["noise"]
    b = e.PT(e.ninv(d))
    if kind == "zd":
        return e.solve(b), e.solve(e.PT(e.ninv(sig + _second_noise(s))))
    x = e.solve(b)
    if kind in ("tts", "batch"):
        return x
    if kind in ("small", "solve64"):
        return b, x
    mu = e.solve(2.0 * (x - _compact_sky(s)) / x.numel())
    gd, gp = e.gradients(d, x, mu)
    return (x, gd, gp) if kind == "grad" else (gd, gp.cpu().numpy(), mu)
