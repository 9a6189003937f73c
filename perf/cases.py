"""What the library's speed is measured on: the calls that a user's program makes, over the sizes
that it makes them at.

A case is one call pattern ("kind") at one size:

  logl   the batched log-likelihood (gwlike.logl), the whole work of a nested sampler's pool
  live   the same with a batch length that the device decides (gwlike.logl_live), as the
         captured slice-sampling moves call it
  grad   log-likelihood and gradient (gwlike.logl_grad, or LogL under autograd), the
         gradient-guided walks and optimisers
  rb     the relative-binning likelihood
  plan   many uneven events in one launch, values and gradients (MultiPlan)

on an event of `ndet` detectors, `duration` seconds, 20 Hz to `f_hi`, optionally with a calibration
model of `nodes` nodes per detector. "fp64" calls take and return float64. A program that asks
for the mixed precision (accurate to about 1e-8 of logL) keeps its walkers, values and gradients
in float32; its calls convert on the way in and out.

Inputs follow the synthetic workloads of the package's synth module: coloured Gaussian noise with
an injected signal, and a batch of prior draws (chirp masses 10 to 60 for black holes, 1 to 1.5
for neutron stars on the 128 s segments, coalescence times within 0.1 s); for relative binning
draws near the fiducial.
"""
from __future__ import annotations

import math
import os

import torch

from paper_1909_11873_amd import gwlike as gw

# launch shapes that the package ships, as its benchmark loads them
gw.autotune_load(os.path.join(os.path.dirname(gw.__file__), "tuning_gfx950.json"))

F_LO = 20.0
BBH = (30.0, 0.8, 0.0, 0.0, 400.0, 2.0, -0.5, 0.6, 1.0, 0.7, 0.0)
BNS = (1.2, 0.8, 0.0, 0.0, 100.0, 2.0, -0.5, 0.6, 1.0, 0.7, 0.0)
# latitude, longitude, x-arm and y-arm azimuth in degrees
SITES = ((46.5, -119.4, 126.0, 36.0), (30.6, -90.8, 198.0, 108.0), (43.6, 10.5, 71.0, 341.0))
MAX_POINT_BINS = 65536 * 16225           # the largest listed batch on its grid


def listed():
    def case(name, kind, ndet, duration, f_hi, batch, precision, nodes=0, bns=False, events=1):
        return {"name": name, "kind": kind, "ndet": ndet, "duration": duration, "f_hi": f_hi, "batch": batch,
                "precision": precision, "nodes": nodes, "bns": bns, "events": events}
    return [
        # one walker of a serial sampler: latency alone
        case("one point", "logl", 1, 4, 1024, 1, "fp64"),
        # a small pool of walkers on a single-detector 4 s segment
        case("small pool", "logl", 1, 4, 1024, 1000, "fp64"),
        # the sampler's shrinkage draws: a partly live batch on the three-detector 8 s segment
        case("slice draws", "live", 3, 8, 2048, 8192, "mixed"),
        # the headline workload: a large batch on the three-detector 8 s segment, both precisions
        case("large batch", "logl", 3, 8, 2048, 65536, "mixed"),
        case("large batch fp64", "logl", 3, 8, 2048, 65536, "fp64"),
        # gradient-guided walkers under autograd, and their float64 form with a ragged size
        case("gradient", "grad", 3, 8, 2048, 16384, "mixed"),
        case("gradient fp64 ragged", "grad", 2, 17, 1613, 3001, "fp64"),
        # a neutron-star segment: 259,585 bins
        case("long segment", "logl", 3, 128, 2048, 4096, "mixed", bns=True),
        # the calibration model, 20 more parameters per detector: values, then gradients
        case("calibrated", "logl", 3, 8, 2048, 16384, "fp64", nodes=10),
        case("calibrated gradient", "grad", 3, 8, 2048, 8192, "mixed", nodes=10),
        # relative binning: a few hundred edges in place of the grid
        case("relative binning", "rb", 3, 8, 2048, 65536, "fp64"),
        # a catalogue of uneven events in one launch, values and gradients
        case("event plan", "plan", 3, 64, 2048, 4096, "fp64", events=12),
    ]


def draw(rng):
    kind = rng.choice(["logl", "logl", "grad", "grad", "live", "rb", "plan"])
    nodes = rng.choice([0, 0, 0, rng.randint(4, 12)]) if kind in ("logl", "grad") else 0
    duration = int(round(math.exp(rng.uniform(math.log(4), math.log(128 if nodes == 0 else 16)))))
    f_hi = rng.choice([1024, 2048, rng.randint(700, 2048)])
    cap = MAX_POINT_BINS // 4 if kind == "plan" or nodes else MAX_POINT_BINS // (2 if kind == "grad" else 1)
    cap = min(65536 if kind != "plan" else 4096, cap // bins(duration, f_hi))
    return {"kind": kind, "ndet": rng.randint(1, 3), "duration": duration, "f_hi": f_hi,
            "batch": int(math.exp(rng.uniform(0.0 if kind in ("logl", "grad") else math.log(200), math.log(cap)))),
            "precision": rng.choice(["mixed", "fp64"]) if kind != "plan" else "fp64", "nodes": nodes,
            "bns": duration >= 64 and rng.random() < 0.7, "events": rng.randint(3, 12) if kind == "plan" else 1}


def bins(duration, f_hi):
    return int(round((f_hi - F_LO) * duration)) + 1


# ---------------------------------------------------------------------------------------------
# The model, in plain torch and float64: injections, and the values that the calls should return.
# ---------------------------------------------------------------------------------------------
T_SUN, C_LIGHT, MPC, R_EARTH, GAMMA_E = 4.925490947641267e-6, 299792458.0, 3.0856775814913673e22, 6.371e6, \
    0.5772156649015329


def _dets(ndet):
    return [tuple(math.radians(x) for x in s) for s in SITES[:ndet]]


def _basis(f):
    x = f ** (1.0 / 3.0)
    lf = torch.log(f)
    return torch.stack([f ** (-5.0 / 3.0), 1.0 / f, x ** -2.0, 1.0 / x, lf, x, x * lf, x * x])


def _point(theta, dets):
    """Phase coefficients [B, 8] over _basis and constant phase [B] (cycles), amplitude [B], per
    detector the complex projection (re, im) and the arrival time [B]."""
    mc, q, s1, s2, dl, ra, dec, inc, psi, phic, tc = theta[:, :11].unbind(1)
    pi = math.pi
    eta = q / (1 + q) ** 2
    mt = mc * eta ** -0.6
    m1, m2 = 1 / (1 + q), q / (1 + q)
    beta = (113 / 12 * m1 ** 2 + 25 / 4 * eta) * s1 + (113 / 12 * m2 ** 2 + 25 / 4 * eta) * s2
    p2 = 3715 / 756 + 55 / 9 * eta
    p3 = -16 * pi + 4 * beta
    p4 = 15293365 / 508032 + 27145 / 504 * eta + 3085 / 72 * eta ** 2 - 395 / 4 * eta * s1 * s2
    p5 = pi * (38645 / 756 - 65 / 9 * eta)
    p6 = 11583231236531 / 4694215680 - 640 / 3 * pi ** 2 - 6848 / 21 * GAMMA_E \
        + (-15737765635 / 3048192 + 2255 / 12 * pi ** 2) * eta + 76055 / 1728 * eta ** 2 - 127825 / 1296 * eta ** 3
    p7 = pi * (77096675 / 254016 + 378515 / 1512 * eta - 74045 / 756 * eta ** 2)
    pm = pi * T_SUN * mt
    lpm, b = torch.log(pm), pm ** (1.0 / 3.0)
    n = 3 / (256 * pi) / eta
    a = torch.stack([n * b ** -5, n * p2 * b ** -3, n * p3 * b ** -2, n * p4 / b, n * p5,
                     n * b * (p6 - 6848 / 21 * (math.log(4.0) + lpm / 3)), n * b * (-6848 / 63), n * p7 * b ** 2], 1)
    c0 = n * p5 * (1 + lpm) - (phic + pi / 4) / (2 * pi)
    amp = math.sqrt(5 / 24) * pi ** (-2 / 3) * (T_SUN * mc) ** (5 / 6) * C_LIGHT / (dl * MPC)
    k = torch.stack([dec.cos() * ra.cos(), dec.cos() * ra.sin(), dec.sin()])
    u = torch.stack([-dec.sin() * ra.cos(), -dec.sin() * ra.sin(), dec.cos()])
    v = torch.stack([-ra.sin(), ra.cos(), torch.zeros_like(ra)])
    x, y = psi.cos() * u + psi.sin() * v, -psi.sin() * u + psi.cos() * v
    proj = []
    for lat, lon, ax, ay in dets:
        north = (-math.sin(lat) * math.cos(lon), -math.sin(lat) * math.sin(lon), math.cos(lat))
        east = (-math.sin(lon), math.cos(lon), 0.0)
        e1 = [math.cos(ax) * n_ + math.sin(ax) * e_ for n_, e_ in zip(north, east)]
        e2 = [math.cos(ay) * n_ + math.sin(ay) * e_ for n_, e_ in zip(north, east)]
        d = torch.tensor([[0.5 * (e1[i] * e1[j] - e2[i] * e2[j]) for j in range(3)] for i in range(3)],
                         dtype=torch.float64, device=theta.device)
        r = (R_EARTH * math.cos(lat) * math.cos(lon), R_EARTH * math.cos(lat) * math.sin(lon),
             R_EARTH * math.sin(lat))
        fp = (x * (d @ x)).sum(0) - (y * (d @ y)).sum(0)
        fx = 2 * (x * (d @ y)).sum(0)
        arrive = tc - (r[0] * k[0] + r[1] * k[1] + r[2] * k[2]) / C_LIGHT
        proj.append((fp * 0.5 * (1 + inc.cos() ** 2), -fx * inc.cos(), arrive))
    return a, c0, amp, proj


def _strain(theta, dets, f):
    """h_det(f) [B, ndet, M]."""
    a, c0, amp, proj = _point(theta, dets)
    phase = a @ _basis(f) + c0[:, None]
    out = []
    for qr, qi, t in proj:
        ph = phase + t[:, None] * f
        ph = -2 * math.pi * (ph - ph.round())
        out.append(amp[:, None] * f ** (-7.0 / 6.0) * torch.complex(qr, qi)[:, None]
                   * torch.complex(ph.cos(), ph.sin()))
    return torch.stack(out, 1)


def _spline_weights(f, n):
    """[M, n]: Catmull-Rom weights in ln f of n nodes, linear ghost nodes beyond the ends."""
    lf = torch.log(f)
    s = ((lf - lf[0]) / ((lf[-1] - lf[0]) / (n - 1))).clamp(0.0, n - 1.0)
    j = s.floor().long().clamp(0, n - 2)
    t = s - j
    w = torch.zeros(f.shape[0], n + 2, dtype=torch.float64, device=f.device)
    cubic = (-t + 2 * t ** 2 - t ** 3, 2 - 5 * t ** 2 + 3 * t ** 3, t + 4 * t ** 2 - 3 * t ** 3, -t ** 2 + t ** 3)
    for i, c in enumerate(cubic):
        w.scatter_add_(1, (j + i)[:, None], 0.5 * c[:, None])
    w[:, 1] += 2 * w[:, 0]
    w[:, 2] -= w[:, 0]
    w[:, n] += 2 * w[:, n + 1]
    w[:, n - 1] -= w[:, n + 1]
    return w[:, 1:n + 1].contiguous()


def _edges(f, eps):
    """Relative-binning edges: where floor(dpsi / eps) changes, and both ends."""
    lo, hi = float(f[0]), float(f[-1])
    d = sum((1.0 if g > 0 else -1.0) * (f / (hi if g > 0 else lo)) ** g for g in (-5 / 3, -2 / 3, 1.0, 5 / 3, 7 / 3))
    cell = torch.floor(2 * math.pi * d / eps)
    at = [0] + (torch.nonzero(cell[1:] != cell[:-1]).reshape(-1) + 1).tolist()
    return at if at[-1] == f.shape[0] - 1 else at + [f.shape[0] - 1]


def _reference(theta, e, grad):
    """(logL, gradient or None) of event inputs `e`, by the definition, a few points at a time."""
    f, df, dets, n = e["f"], e["df"], e["dets"], e["nodes"]
    amp_f = f ** (-7.0 / 6.0)
    u = 4 * df * amp_f * e["data"].conj() / e["psd"]                         # [ndet, M]
    kd = 4 * df * amp_f ** 2 / e["psd"]
    if e["fiducial"] is not None:
        at = torch.tensor(_edges(f, 0.1), device=f.device)
        h0 = _strain(e["fiducial"], dets, f)[0]
        h0 = h0 / amp_f
        fe = f[at]
        c = u * h0
        g = torch.bucketize(f, fe, right=True).clamp(1, len(at) - 1) - 1      # span of every bin
        t = (f - fe[g]) / (fe[g + 1] - fe[g])
        summ = torch.zeros(len(dets), len(at), dtype=torch.complex128, device=f.device)
        summ.index_add_(1, g, c * (1 - t))
        summ.index_add_(1, g + 1, c * t)
        u, f = summ / h0[:, at], fe
    basis = _basis(f)
    w = _spline_weights(f, n) if n else None
    step = max(1, int(2.4e7) // f.shape[0])
    val, gr = [], []
    for i in range(0, theta.shape[0], step):
        th = theta[i:i + step].clone().requires_grad_(grad)
        with torch.set_grad_enabled(grad):
            a, c0, amp, proj = _point(th, dets)
            phase = a @ basis + c0[:, None]
            tot = 0.0
            for d, (qr, qi, t) in enumerate(proj):
                ph = phase + t[:, None] * f
                ph = -2 * math.pi * (ph - ph.detach().round())
                gain = 1.0
                if n:
                    at = 11 + 2 * n * d
                    gain = 1 + th[:, at:at + n] @ w.T
                    ph = ph + th[:, at + n:at + 2 * n] @ w.T
                cs, sn = gain * ph.cos(), gain * ph.sin()
                zr, zi = cs @ u[d].real - sn @ u[d].imag, cs @ u[d].imag + sn @ u[d].real
                norm = (gain ** 2) @ kd[d] if n else kd[d].sum()
                tot = tot + amp * (qr * zr - qi * zi) - 0.5 * amp ** 2 * (qr ** 2 + qi ** 2) * norm
        val.append(tot.detach())
        if grad:
            gr.append(torch.autograd.grad(tot.sum(), th)[0])
    return torch.cat(val), torch.cat(gr) if grad else None


# ---------------------------------------------------------------------------------------------
def _event_inputs(case, gen, duration, bns, rb=False):
    dev = torch.device("cuda:0")
    m = bins(duration, case["f_hi"])
    df = (case["f_hi"] - F_LO) / (m - 1)
    f = F_LO + df * torch.arange(m, dtype=torch.float64, device=dev)
    x = f / 215.0
    s = 1e-49 * (x ** -4.14 - 5.0 * x ** -2 + 111.0 * (1.0 - x ** 2 + 0.5 * x ** 4) / (1.0 + 0.5 * x ** 2))
    dets = _dets(case["ndet"])
    psd = s.repeat(len(dets), 1)
    noise = torch.randn(len(dets), m, 2, dtype=torch.float64, device=dev, generator=gen)
    theta0 = torch.tensor([BNS if bns else BBH], dtype=torch.float64, device=dev)
    data = torch.sqrt(psd / (4.0 * df)) * torch.view_as_complex(noise) + _strain(theta0, dets, f)[0]
    return {"f": f, "df": df, "psd": psd, "data": data, "dets": dets, "nodes": case["nodes"],
            "fiducial": theta0 if rb else None}


def _points(e, n, gen, bns):
    dev = torch.device("cuda:0")
    u = torch.rand(n, 11, dtype=torch.float64, device=dev, generator=gen)
    if e["fiducial"] is not None:
        scale = torch.tensor([0.05, 0.05, 0.1, 0.1, 40.0, 0.05, 0.05, 0.1, 0.2, 0.5, 2e-3], dtype=torch.float64,
                             device=dev)
        th = e["fiducial"] + scale * (2 * u - 1)
    else:
        lo, hi = (1.0, 1.5) if bns else (10.0, 60.0)
        th = torch.stack([lo + (hi - lo) * u[:, 0], 0.2 + 0.8 * u[:, 1], -0.9 + 1.8 * u[:, 2], -0.9 + 1.8 * u[:, 3],
                          (1e6 + u[:, 4] * (8e9 - 1e6)) ** (1.0 / 3.0), 2 * math.pi * u[:, 5],
                          torch.asin(2 * u[:, 6] - 1), torch.acos(2 * u[:, 7] - 1), math.pi * u[:, 8],
                          2 * math.pi * u[:, 9], -0.1 + 0.2 * u[:, 10]], 1)
    if e["nodes"]:
        c = 0.05 * torch.randn(n, 2 * e["nodes"] * len(e["dets"]), dtype=torch.float64, device=dev, generator=gen)
        th = torch.cat([th, c], 1)
    return th.contiguous()


def _plan_sizes(case):
    """(duration, batch) of every event of a plan, uneven, up to the case's own."""
    e = case["events"]
    return [(max(4, int(case["duration"] * 16.0 ** (-(j * 5 % e) / e))),
             max(1, int(case["batch"] * 16.0 ** (-(j * 7 % e) / e)))) for j in range(e)]


def _inputs(case, seed):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    sizes = _plan_sizes(case) if case["kind"] == "plan" else [(case["duration"], case["batch"])]
    es = [_event_inputs(case, gen, t, case["bns"], case["kind"] == "rb") for t, _ in sizes]
    ths = [_points(e, b, gen, case["bns"]) for e, (_, b) in zip(es, sizes)]
    if case["precision"] == "mixed":
        ths = [t.float() for t in ths]
    return es, ths


def _live(case):
    return max(1, case["batch"] * 2 // 5)


def prepare(case, seed):
    es, ths = _inputs(case, seed)
    evs = [gw.Event(e["data"], e["psd"], e["dets"], e["f"], e["df"], calibration_nodes=e["nodes"],
                    fiducial=None if e["fiducial"] is None else e["fiducial"][0].tolist()) for e in es]
    s = {"kind": case["kind"], "precision": case["precision"], "event": evs[0], "theta": ths[0]}
    if case["kind"] == "plan":
        s |= {"plan": gw.MultiPlan(evs, [len(t) for t in ths], case["precision"], True), "events": evs, "thetas": ths}
    if case["kind"] == "live":
        s |= {"live": torch.tensor(_live(case), dtype=torch.int64, device="cuda:0"),
              "out": torch.zeros(case["batch"], dtype=torch.float64, device="cuda:0")}
    if case["kind"] == "grad" and case["precision"] == "mixed":
        s["theta"].requires_grad_(True)
    return s


def run(s):
    kind, prec, theta = s["kind"], s["precision"], s["theta"]
    if kind == "plan":
        val, grad, _ = s["plan"].launch(s["thetas"])
        return {"logl": val, "grad": grad}
    if kind == "grad":
        if prec == "fp64":
            val, grad = gw.logl_grad(theta, s["event"], prec)
            return {"logl": val, "grad": grad}
        val = gw.LogL.apply(theta.double(), s["event"], prec)          # walkers in float32, under autograd
        grad, = torch.autograd.grad(val.sum(), theta)
        return {"logl": val.detach().float(), "grad": grad}
    if prec == "mixed":
        theta = theta.double()
    if kind == "live":
        val = gw.logl_live(theta, s["live"], s["event"], prec, out=s["out"])
    else:
        val = gw.logl(theta, s["event"], prec)
    return {"logl": val.float() if prec == "mixed" else val}


def exact(case, seed):
    es, ths = _inputs(case, seed)
    grad = case["kind"] in ("grad", "plan")
    if sum(len(t) * e["f"].shape[0] * len(e["dets"]) for e, t in zip(es, ths)) > 4e9:
        return None
    got = []
    for e, t in zip(es, ths):
        t = t.double()
        if case["kind"] == "live":
            val = torch.zeros(len(t), dtype=torch.float64, device=t.device)
            val[:_live(case)] = _reference(t[:_live(case)], e, False)[0]
            got.append((val, None))
        else:
            got.append(_reference(t, e, grad))
    if case["kind"] == "plan":
        return {"logl": [v for v, _ in got], "grad": [g for _, g in got]}
    return {"logl": got[0][0], "grad": got[0][1]} if grad else {"logl": got[0][0]}


def work(case):
    """One pass's least work. Bytes: the points in, the whitened data once, the values (and gradient)
    out. Operations: the model is a short chirp, so the sum over the bins of a segment is one over
    as many samples as the chirp's time-frequency area holds (2 x the integral of its largest
    |t(f)| over the band, at most the bins themselves; relative binning: about 300 edges); per
    sample 40 for the phase and the phasor and 8 per detector for the complex multiply-add, twice
    that with the gradient."""
    sizes = _plan_sizes(case) if case["kind"] == "plan" else [(case["duration"], case["batch"])]
    nd, grad = case["ndet"], case["kind"] in ("grad", "plan")
    cols = 11 + 2 * case["nodes"] * nd
    width = 4 if case["precision"] == "mixed" else 8
    mc = 1.0 if case["bns"] else 10.0
    tau = 5.0 / 256.0 * (mc * T_SUN) ** (-5.0 / 3.0) * (math.pi * F_LO) ** (-8.0 / 3.0)
    samples = 2.0 * (0.121 * (case["f_hi"] - F_LO) + 0.6 * tau * F_LO)
    nbytes = flops = 0.0
    for duration, batch in sizes:
        m = bins(duration, case["f_hi"])
        live = _live(case) if case["kind"] == "live" else batch
        n = 300 if case["kind"] == "rb" else min(m, samples)
        nbytes += 16.0 * nd * m + live * width * (cols + 1 + (cols if grad else 0))
        flops += live * n * (40.0 + 8.0 * nd) * (2 if grad else 1)
    return {"bytes": nbytes, "flops": flops}
