"""Band-limited rows against the sum over every bin.

A group of 64 points whose chirps stay inside a band of arrival times walks a few hundred
band-limited rows in place of the grid's bins; a launch whose chunks hold at most 20 bins walks the
bins. Two launch layouts of the same event therefore compare the two sums directly. The rows
reproduce each bin's phasor to about 1e-14 (1e-13 in the worst chirp at a panel's edge), so a point's
values differ by at most 1e-13 sum_k |A Q u_k| <= 1e-13 |h| |d| (norms of signal and data in the noise-weighted
inner product), and its gradient by the same share of its scale.
"""
import json
import math
import os

import numpy as np
import pytest
import torch

from oracle import gw_oracle as o
from paper_1909_11873_amd import gwlike as gw
from paper_1909_11873_amd import synth
from tests.helpers import event_inputs, scaled_grad_error

DEV = torch.device("cuda:0")
CACHE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1909_11873_amd",
                     "tuning_gfx950.json")


@pytest.mark.parametrize("sigma", [1.25, 1.4, 1.6, 2.0, 2.5, 3.0])
def test_windowed_sinc_reproduces_tones_of_its_band(sigma):
    """The rows' kernel, from its definition: a tone of any time within the band, anywhere between two
    rows, to 2e-14; a tone beyond the band's far side (the first alias) is not reproduced."""
    w = math.ceil(292.0 / (2.285 * 2.0 * math.pi * (1.0 - 1.0 / sigma)))
    beta = 0.98 * math.pi * 0.5 * w * (1.0 - 1.0 / sigma)
    x = np.linspace(0.0, 1.0, 33)[:, None] - np.arange(-(w // 2) - 1, w // 2 + 3)[None, :]
    r2 = 1.0 - (2.0 * x / w) ** 2
    k = np.where(r2 > 0, np.sinc(x) * np.exp(beta * (np.sqrt(np.maximum(r2, 0.0)) - 1.0)), 0.0)
    for nu in np.linspace(-0.5 / sigma, 0.5 / sigma, 41):       # cycles per row
        got = k @ np.exp(-2j * np.pi * nu * np.arange(-(w // 2) - 1, w // 2 + 3))
        assert np.abs(got - np.exp(-2j * np.pi * nu * np.linspace(0.0, 1.0, 33))).max() <= 2e-14
    alias = k @ np.exp(-2j * np.pi * (1.0 - 0.5 / sigma) * np.arange(-(w // 2) - 1, w // 2 + 3))
    assert np.abs(alias - np.exp(-2j * np.pi * (1.0 - 0.5 / sigma) * np.linspace(0.0, 1.0, 33))).max() > 0.5


def _layout(path, nd, M, prec, grad, batch, waves, groups, setup):
    npg = (batch + 63) // 64
    entry = {"ndet": nd, "mixed": int(prec == "mixed"), "grad": int(grad), "M": M,
             "npg_bucket": 1 << (npg - 1).bit_length(), "waves": waves, "groups": groups, "setup": setup,
             "sepepi": 0, "ms": 1.0}
    with open(path, "w") as fh:
        fh.write('{"arch": "gfx950", "entries": [\n  ' + json.dumps(entry) + "\n]}\n")
    gw.autotune_load(path)


def _points(kind, n, seed):
    rng = np.random.default_rng(seed)
    th = synth.prior_draw(rng, n, mc_range=(1.0, 1.5) if kind == "light" else (10.0, 60.0))
    if kind == "late":                    # arrival times spread beyond every band around zero
        th[:, 10] = rng.uniform(-6.0, 6.0, n)
    if kind == "wide":                    # most groups in the widest bands
        th[:, 10] = rng.uniform(-0.3, 0.3, n)
    if kind == "narrow":                  # a converged sampler's batch
        th[:, 10] = rng.uniform(-1e-3, 1e-3, n)
    if kind == "invalid":                 # NaN rows and a far outlier among ordinary points
        th[3, 1] = 1.5
        th[70, 10] = 1e9
        th[130:194, 1] = -1.0             # a whole group
    return th


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["prior", "late", "wide", "narrow", "light", "invalid"])
@pytest.mark.parametrize("nd,duration,f_lo,f_hi,uniform", [
    (3, 8.0, 20.0, 1024.0, True), (2, 17.0, 20.0, 611.0, True), (1, 4.0, 11.0, 1024.0, True),
    (3, 8.0, 20.0, 400.0, False), (2, 32.0, 20.0, 500.0, True)])
def test_rows_match_every_bin(kind, nd, duration, f_lo, f_hi, uniform, tmp_path):
    df = 1.0 / duration
    f = synth.freq_grid(f_lo, f_hi, df)
    if not uniform:                       # increasing, with steps between 0.6 and 1.4 of the mean
        f = f + 0.2 * df * np.sin(np.arange(len(f)) * 1.7)
    M = len(f)
    psd = np.stack([synth.psd_fit(f)] * nd)
    dets = np.array([synth.detector_rad(n) for n in ("D1", "D2", "D3")[:nd]])
    data = np.stack([synth.noise(900 + i, psd[i], df) for i in range(nd)]) + o.strain_all(synth.THETA0_BBH, dets, f).numpy()
    th = _points(kind, 257, 5)
    if kind != "invalid":
        th[0] = synth.THETA0_BBH
    t = torch.tensor(th, device=DEV)
    ev = gw.Event(torch.tensor(data, device=DEV), torch.tensor(psd, device=DEV), dets, torch.tensor(f, device=DEV), df)
    path = str(tmp_path / "layout.json")
    groups = -(-M // (16 * 20))           # 16 wavefronts x groups: chunks of at most 20 bins
    dn = math.sqrt(sum(float((4 * df * np.abs(d) ** 2 / s).sum()) for d, s in zip(data, psd)))
    try:
        for prec in ("fp64", "mixed"):
            for grad in (False, True):
                got = []
                for waves, grp, setup in ((16, groups, 0), (4, 1, 0), (16, 3, 1), (1, 2, 1)):
                    _layout(path, nd, M, prec, grad, len(th), waves, grp, setup)
                    v, g = gw.logl_grad(t, ev, prec) if grad else (gw.logl(t, ev, prec), torch.zeros(len(th), 11))
                    got.append((v.cpu().numpy(), g.cpu().numpy()))
                bins, gbins = got[0]
                ok = np.isfinite(bins)
                beyond = 1e9 * f[-1] >= 2.0 ** 39   # the outlier's phase: outside the range that is evaluated
                assert ok.sum() == (257 - 65 - beyond if kind == "invalid" else 257)
                # |h|^2 <= 2 (<d|h> - logL) <= ..., bounded from logL = <d|h> - |h|^2 / 2 and <d|h> <= |d| |h|
                hn = dn + np.sqrt(np.maximum(dn ** 2 - 2.0 * bins[ok], 0.0))
                tol = 1e-13 * hn * dn + 1e-9 if prec == "fp64" else 1e-3
                for v, g in got[1:]:
                    assert np.array_equal(np.isfinite(v), ok)
                    err = np.abs(v[ok] - bins[ok])
                    assert (err <= tol).all(), (prec, grad, err.max())
                    if grad:
                        e = scaled_grad_error(g[ok], gbins[ok])
                        assert e.max() <= (2e-9 if prec == "fp64" else 1e-3), (prec, e.max())
    finally:
        ev.close()
        gw.autotune_load(CACHE)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("grad", [False, True])
def test_plan_of_events_matches_every_bin(prec, grad, tmp_path):
    """Groups that walk rows and groups that walk bins in one plan (points near the origin, spread over
    the segment, and invalid ones; a short grid, an empty batch): the values and gradients of single
    calls that walk every bin, the same bits on a second launch, in both queue orders."""
    events, thetas, want = [], [], []
    path = str(tmp_path / "layout.json")
    try:
        for kind, f_hi, n in (("prior", 700.0, 200), ("late", 300.0, 129), ("invalid", 611.0, 257), ("light", 40.0, 64),
                              ("prior", 300.0, 0)):
            spec, f, psd, data, dets = event_inputs(1, f_hi=f_hi)
            t = torch.tensor(_points(kind, max(n, 257), 8)[:n], device=DEV)
            ev = gw.Event(torch.tensor(data, device=DEV), torch.tensor(psd, device=DEV), dets,
                          torch.tensor(f, device=DEV), spec.df)
            if n:
                _layout(path, 3, len(f), prec, grad, n, 16, -(-len(f) // 320), 0)
                want.append(gw.logl_grad(t, ev, prec) if grad else (gw.logl(t, ev, prec), None))
            else:
                want.append((torch.empty(0), torch.empty(0, 11)))
            events.append(ev)
            thetas.append(t)
        got = []
        for order in ("ascending", "descending"):
            plan = gw.MultiPlan(events, [len(t) for t in thetas], prec, with_grad=grad, order=order)
            for _ in range(2):
                v, g, _ = plan.launch(thetas)
                got.append([x.cpu().numpy() for x in v] + ([x.cpu().numpy() for x in g] if grad else []))
            plan.close()
        for other in got[1:]:
            assert all(np.array_equal(a, b, equal_nan=True) for a, b in zip(got[0], other))
        for i, (v, g) in enumerate(want):
            v = v.cpu().numpy()
            ok = np.isfinite(v)
            assert np.array_equal(np.isfinite(got[0][i]), ok)
            assert (np.abs(got[0][i][ok] - v[ok]) <= (1e-7 if prec == "fp64" else 1e-3)).all()
            if grad and len(v):
                e = scaled_grad_error(got[0][len(want) + i][ok], g.cpu().numpy()[ok])
                assert e.max() <= (2e-9 if prec == "fp64" else 1e-3), e.max()
    finally:
        gw.autotune_load(CACHE)


@pytest.mark.gpu
def test_grids_without_bands_keep_their_bins():
    """Grids that are not increasing, or too short to have bands, give the oracle's values as before."""
    for f_hi, flip in ((300.0, True), (30.0, False)):
        spec, f, psd, data, dets = event_inputs(1, f_hi=f_hi)
        if flip:                          # the same bins in descending order
            f, psd, data = f[::-1].copy(), psd[:, ::-1].copy(), data[:, ::-1].copy()
        th = synth.theta_batch(spec, 5)
        ev = gw.Event(torch.tensor(data, device=DEV), torch.tensor(psd, device=DEV), dets, torch.tensor(f, device=DEV),
                      spec.df)
        ref = o.logl(th, data, psd, dets, f, spec.df).numpy()
        for prec, tol in (("fp64", 1e-6), ("mixed", 1e-3)):
            assert np.abs(gw.logl(torch.tensor(th, device=DEV), ev, prec).cpu().numpy() - ref).max() <= tol
        ev.close()


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["prior", "late", "wide", "light", "invalid"])
@pytest.mark.parametrize("nd,nodes,sigma,f_hi", [(3, 10, 0.05, 700.0), (2, 4, 0.5, 400.0), (1, 16, 0.2, 1024.0)])
def test_calibrated_rows_match_every_bin(kind, nd, nodes, sigma, f_hi):
    """The calibrated loop on rows, which keep to the spline's node intervals, against the same bins with
    two neighbours swapped: such a grid does not increase, so it has no rows. Node values up to half a
    radian (a phase slope that widens the arrival times), values and all gradients."""
    spec, f, psd, data, dets = event_inputs(1, f_hi=f_hi, ndet=nd)
    k = len(f) // 2
    order = np.r_[0:k, k + 1, k, k + 2:len(f)]
    mk = lambda i: gw.Event(torch.tensor(np.ascontiguousarray(data[:, i]), device=DEV),
                            torch.tensor(np.ascontiguousarray(psd[:, i]), device=DEV), dets,
                            torch.tensor(f[i], device=DEV), spec.df, calibration_nodes=nodes)
    ev, plain = mk(np.arange(len(f))), mk(order)
    th = _points(kind, 257, 11)
    rng = np.random.default_rng(12)
    th = np.concatenate([th, sigma * rng.standard_normal((len(th), 2 * nodes * nd))], axis=1)
    t = torch.tensor(th, device=DEV)
    dn = math.sqrt(sum(float((4 * spec.df * np.abs(d) ** 2 / s).sum()) for d, s in zip(data, psd)))
    for prec in ("fp64", "mixed"):
        want = gw.logl(t, plain, prec).cpu().numpy()
        ok = np.isfinite(want)
        hn = dn + np.sqrt(np.maximum(dn ** 2 - 2.0 * want[ok], 0.0))
        tol = 1e-13 * hn * dn + 1e-9 if prec == "fp64" else 1e-3
        got = gw.logl(t, ev, prec).cpu().numpy()
        assert np.array_equal(np.isfinite(got), ok)
        assert (np.abs(got[ok] - want[ok]) <= tol).all(), (prec, np.abs(got[ok] - want[ok]).max())
        v, g = (x.cpu().numpy() for x in gw.logl_grad(t, ev, prec))
        vw, gw_ = (x.cpu().numpy() for x in gw.logl_grad(t, plain, prec))
        assert np.array_equal(np.isfinite(v), ok) and np.array_equal(np.isfinite(g), np.isfinite(gw_))
        assert (np.abs(v[ok] - want[ok]) <= tol).all()
        e = scaled_grad_error(g[ok][:, :11], gw_[ok][:, :11])
        c = np.abs(g[ok][:, 11:] - gw_[ok][:, 11:]) / np.abs(gw_[ok][:, 11:]).max(axis=1, keepdims=True)
        lim = 2e-9 if prec == "fp64" else 1e-3
        assert e.max() <= lim and c.max() <= lim, (prec, e.max(), c.max())
    ev.close()
    plain.close()


@pytest.mark.gpu
@pytest.mark.parametrize("kind,n", [("prior", 16384), ("prior", 17473), ("late", 16385), ("invalid", 16448),
                                    ("same", 16385)])
@pytest.mark.parametrize("nodes", [0, 5])
def test_ordered_points_match_small_calls(kind, n, nodes):
    """A large call takes its points in an order of its own, a call of 1,000 in the caller's: other groups
    and so other rows, each within the rows' error of the bins. Every value and gradient belongs to its
    point; points alike in mass and time, infinite ones and a last block of one point included."""
    spec, f, psd, data, dets = event_inputs(1, f_hi=300.0, ndet=2)
    ev = gw.Event(torch.tensor(data, device=DEV), torch.tensor(psd, device=DEV), dets, torch.tensor(f, device=DEV),
                  spec.df, calibration_nodes=nodes)
    th = _points("prior" if kind == "same" else kind, n, 21)
    rng = np.random.default_rng(22)
    if kind == "same":
        th[:, 0], th[:, 10] = 30.0, 0.01
        th[5, 10], th[6, 0], th[7, 10] = np.inf, np.nan, 1e300
    if nodes:
        th = np.concatenate([th, 0.05 * rng.standard_normal((n, 2 * nodes * 2))], axis=1)
    t = torch.tensor(th, device=DEV)
    dn = math.sqrt(sum(float((4 * spec.df * np.abs(d) ** 2 / s).sum()) for d, s in zip(data, psd)))
    for prec in ("fp64", "mixed"):
        want, gwant = (torch.cat(x).cpu().numpy() for x in
                       zip(*(gw.logl_grad(t[i:i + 1000].contiguous(), ev, prec) for i in range(0, n, 1000))))
        ok = np.isfinite(want)
        hn = dn + np.sqrt(np.maximum(dn ** 2 - 2.0 * want[ok], 0.0))
        tol = 2e-13 * hn * dn + 2e-9 if prec == "fp64" else 2e-3
        v, g = (x.cpu().numpy() for x in gw.logl_grad(t, ev, prec))
        for got in (gw.logl(t, ev, prec).cpu().numpy(), v):
            assert np.array_equal(np.isfinite(got), ok)
            assert (np.abs(got[ok] - want[ok]) <= tol).all(), (prec, np.abs(got[ok] - want[ok]).max())
        assert np.array_equal(np.isfinite(g), np.isfinite(gwant))
        lim = 2e-9 if prec == "fp64" else 1e-3
        assert scaled_grad_error(g[ok][:, :11], gwant[ok][:, :11]).max() <= lim
        if nodes:
            c = np.abs(g[ok][:, 11:] - gwant[ok][:, 11:]) / np.abs(gwant[ok][:, 11:]).max(axis=1, keepdims=True)
            assert c.max() <= lim
    ev.close()


@pytest.mark.gpu
def test_capture_without_room_for_the_order():
    """On a capturing stream whose workspace is too small for the points' order a large call keeps the
    caller's order, as it needs no workspace otherwise; each replay gives the eager call's values."""
    spec, f, psd, data, dets = event_inputs(1, f_hi=120.0, ndet=1)
    ev = gw.Event(torch.tensor(data, device=DEV), torch.tensor(psd, device=DEV), dets, torch.tensor(f, device=DEV),
                  spec.df)
    n = 600000
    t = torch.tensor(_points("prior", 4096, 31), device=DEV).repeat(-(-n // 4096), 1)[:n].contiguous()
    want = gw.logl(t, ev, "fp64")
    out = torch.empty_like(want)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        gw.logl(t[:64].contiguous(), ev, "fp64")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        out.copy_(gw.logl(t, ev, "fp64"))
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        ok = torch.isfinite(want)
        assert torch.equal(torch.isfinite(out), ok)
        scale = float(want[ok].abs().max())
        assert float((out[ok] - want[ok]).abs().max()) <= 1e-11 * scale + 2e-9
    ev.close()


@pytest.mark.gpu
@pytest.mark.parametrize("lo,hi", [(0.07, 0.11), (-0.13, -0.09), (0.125, 0.16)])
@pytest.mark.parametrize("nodes", [0, 8])
def test_bands_off_the_centre(lo, hi, nodes):
    """Groups of heavy systems that arrive within 40 ms of one another, away from zero, take the bands
    centred near them; against the same bins with two neighbours swapped, which have no rows."""
    spec, f, psd, data, dets = event_inputs(1, f_hi=900.0)
    k = len(f) // 2
    swap = np.r_[0:k, k + 1, k, k + 2:len(f)]
    mk = lambda i: gw.Event(torch.tensor(np.ascontiguousarray(data[:, i]), device=DEV),
                            torch.tensor(np.ascontiguousarray(psd[:, i]), device=DEV), dets,
                            torch.tensor(f[i], device=DEV), spec.df, calibration_nodes=nodes)
    ev, plain = mk(np.arange(len(f))), mk(swap)
    rng = np.random.default_rng(41)
    th = synth.prior_draw(rng, 200, mc_range=(40.0, 60.0))
    th[:, 10] = rng.uniform(lo, hi, len(th))
    if nodes:
        th = np.concatenate([th, 0.05 * rng.standard_normal((len(th), 2 * nodes * 3))], axis=1)
    t = torch.tensor(th, device=DEV)
    dn = math.sqrt(sum(float((4 * spec.df * np.abs(d) ** 2 / s).sum()) for d, s in zip(data, psd)))
    for prec in ("fp64", "mixed"):
        want, gwant = (x.cpu().numpy() for x in gw.logl_grad(t, plain, prec))
        hn = dn + np.sqrt(np.maximum(dn ** 2 - 2.0 * want, 0.0))
        tol = 1e-13 * hn * dn + 1e-9 if prec == "fp64" else 1e-3
        v, g = (x.cpu().numpy() for x in gw.logl_grad(t, ev, prec))
        for got in (v, gw.logl(t, ev, prec).cpu().numpy()):
            assert (np.abs(got - want) <= tol).all(), (prec, np.abs(got - want).max())
        assert scaled_grad_error(g[:, :11], gwant[:, :11]).max() <= (2e-9 if prec == "fp64" else 1e-3)
    ev.close()
    plain.close()


@pytest.mark.gpu
@pytest.mark.parametrize("batch,live", [(65, 64), (8192, 1), (8192, 3277), (33000, 32769), (33000, 0)])
def test_live_calls_on_rows(batch, live):
    """Live-length calls over their range of workgroups per group, many to one: the live points' values,
    to the rows' error, and no other written."""
    spec, f, psd, data, dets = event_inputs(1, f_hi=700.0)
    ev = gw.Event(torch.tensor(data, device=DEV), torch.tensor(psd, device=DEV), dets, torch.tensor(f, device=DEV),
                  spec.df)
    t = torch.tensor(_points("prior", 4096, 51), device=DEV).repeat(-(-batch // 4096), 1)[:batch].contiguous()
    dn = math.sqrt(sum(float((4 * spec.df * np.abs(d) ** 2 / s).sum()) for d, s in zip(data, psd)))
    want = gw.logl(t[:1000].contiguous(), ev, "fp64")
    out = torch.full((batch,), -1.0, dtype=torch.float64, device=DEV)
    gw.logl_live(t, torch.tensor(live, dtype=torch.int64, device=DEV), ev, "fp64", out=out)
    n = min(live, 1000)
    w = want[:n].cpu().numpy()[:min(n, batch)]
    hn = dn + np.sqrt(np.maximum(dn ** 2 - 2.0 * w, 0.0))
    assert (np.abs(out[:len(w)].cpu().numpy() - w) <= 2e-13 * hn * dn + 2e-9).all()
    assert bool((out[live:] == -1.0).all()) and bool((out[:live] != -1.0).all())
    ev.close()


@pytest.mark.gpu
@pytest.mark.parametrize("nodes,f_lo,f_hi,duration,sigma", [
    (16, 20.0, 60.0, 256.0, 0.1), (16, 30.0, 120.0, 128.0, 0.1), (16, 20.0, 200.0, 8.0, 0.3), (12, 20.0, 700.0, 8.0, 0.1)])
def test_calibrated_rows_on_narrow_bands(nodes, f_lo, f_hi, duration, sigma):
    """Node spacings of 0.07 to 0.3 in ln f, every group of 64 points one point: nothing but the bound on the
    calibration phase's slope widens the group's arrival times. Against the same bins with two neighbours
    swapped, which have no rows; bounds as for other calibrated rows."""
    df = 1.0 / duration
    f = synth.freq_grid(f_lo, f_hi, df)
    psd = synth.psd_fit(f)[None]
    dets = np.array([synth.detector_rad("D1")])
    data = synth.noise(77, psd[0], df)[None] + o.strain_all(synth.THETA0_BBH, dets, f).numpy()
    k = len(f) // 2
    swap = np.r_[0:k, k + 1, k, k + 2:len(f)]
    mk = lambda i: gw.Event(torch.tensor(np.ascontiguousarray(data[:, i]), device=DEV),
                            torch.tensor(np.ascontiguousarray(psd[:, i]), device=DEV), dets,
                            torch.tensor(f[i], device=DEV), df, calibration_nodes=nodes)
    ev, plain = mk(np.arange(len(f))), mk(swap)
    rng = np.random.default_rng(61)
    th = synth.prior_draw(rng, 24, mc_range=(20.0, 60.0))
    th = np.repeat(np.concatenate([th, sigma * rng.standard_normal((24, 2 * nodes))], axis=1), 64, axis=0)
    t = torch.tensor(th, device=DEV)
    dn = math.sqrt(float((4 * df * np.abs(data) ** 2 / psd).sum()))
    want, gwant = (x.cpu().numpy() for x in gw.logl_grad(t, plain, "fp64"))
    hn = dn + np.sqrt(np.maximum(dn ** 2 - 2.0 * want, 0.0))
    v, g = (x.cpu().numpy() for x in gw.logl_grad(t, ev, "fp64"))
    for got in (v, gw.logl(t, ev, "fp64").cpu().numpy()):
        assert (np.abs(got - want) <= 1e-13 * hn * dn + 1e-9).all(), (np.abs(got - want) / (hn * dn)).max()
    c = np.abs(g[:, 11:] - gwant[:, 11:]) / np.abs(gwant[:, 11:]).max(axis=1, keepdims=True)
    assert scaled_grad_error(g[:, :11], gwant[:, :11]).max() <= 2e-9 and c.max() <= 2e-9
    ev.close()
    plain.close()


def _both(cfg, nodes, f_hi, nd):
    """An event and the same bins with two neighbours swapped, which have no rows; |d|."""
    spec, f, psd, data, dets = event_inputs(cfg, f_hi=f_hi, ndet=nd)
    k = len(f) // 2
    swap = np.r_[0:k, k + 1, k, k + 2:len(f)]
    mk = lambda i: gw.Event(torch.tensor(np.ascontiguousarray(data[:, i]), device=DEV),
                            torch.tensor(np.ascontiguousarray(psd[:, i]), device=DEV), dets,
                            torch.tensor(f[i], device=DEV), spec.df, calibration_nodes=nodes)
    dn = math.sqrt(sum(float((4 * spec.df * np.abs(d) ** 2 / s).sum()) for d, s in zip(data, psd)))
    return mk(np.arange(len(f))), mk(swap), len(f), dn


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("grad", [False, True])
@pytest.mark.parametrize("nodes", [0, 6])
@pytest.mark.parametrize("n", [257, 20000])
def test_which_calls_walk_rows(prec, grad, nodes, n):
    """What the comparisons of rows with bins rest on: points near the origin walk far fewer rows than bins, in
    float64; points all over the segment the bins, in the call's precision (in a large call's order a group holds a
    part of them, and may still find rows); an event without rows every bin."""
    ev, plain, M, _ = _both(1, nodes, 1024.0, 3)
    for kind, most in (("prior", 0.35), ("narrow", 0.3), ("wide", 0.8), ("late", 1.0)):
        th = _points("narrow" if kind == "narrow" else kind, n, 5)
        if nodes:
            th = np.concatenate([th, 0.05 * np.random.default_rng(1).standard_normal((n, 6 * nodes))], axis=1)
        t = torch.tensor(th, device=DEV)
        rows, bins = gw.call_rows(t, ev, prec, grad)
        if kind == "late" and n > 16384:
            assert 0.9 * n * M < rows + bins <= n * M
        elif kind == "late":
            assert (rows, bins) == ((n * M, 0) if prec == "fp64" else (0, n * M))
        else:
            assert bins == 0 and 100 * n < rows < most * n * M, (kind, rows / (n * M), bins)
        assert gw.call_rows(t, plain, prec, grad) == ((n * M, 0) if prec == "fp64" else (0, n * M))
    ev.close()
    plain.close()


@pytest.mark.gpu
@pytest.mark.parametrize("nodes", [0, 6])
@pytest.mark.parametrize("mass", [12.0, 60.0])
def test_bands_up_to_their_limits(mass, nodes):
    """Groups of one point each, whose arrival times step by a millisecond from -0.35 to 0.65 s: some reach each
    band's limit to within a hundredth of its half-width before the next one takes over."""
    ev, plain, M, dn = _both(1, nodes, 700.0, 2)
    th = np.repeat(synth.THETA0_BBH[None], 1024, axis=0)
    th[:, 0] = mass
    th[:, 10] = -0.35 + 1e-3 * np.arange(1024)
    if nodes:
        th = np.concatenate([th, 0.1 * np.random.default_rng(3).standard_normal((1024, 4 * nodes))], axis=1)
    sizes = set()
    for i in range(0, 1024, 100):
        t = torch.tensor(np.repeat(th[i:i + 100], 64, axis=0), device=DEV)
        want, gwant = (x.cpu().numpy() for x in gw.logl_grad(t, plain, "fp64"))
        v, g = (x.cpu().numpy() for x in gw.logl_grad(t, ev, "fp64"))
        hn = dn + np.sqrt(np.maximum(dn ** 2 - 2.0 * want, 0.0))
        for got in (v, gw.logl(t, ev, "fp64").cpu().numpy()):
            assert (np.abs(got - want) <= 1e-13 * hn * dn + 1e-9).all(), (np.abs(got - want) / (hn * dn)).max()
        assert scaled_grad_error(g[:, :11], gwant[:, :11]).max() <= 2e-9
        for j in range(0, 100, 9):
            sizes.add(gw.call_rows(t[64 * j:64 * j + 64], ev, "fp64", True)[0])
    assert len(sizes) >= 10                                    # many bands took their turn
    ev.close()
    plain.close()
