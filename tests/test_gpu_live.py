"""gwl_logl_batch_live (a batch whose length the device decides): the first *live points come out
bit for bit as in the same call with every point live, and within rounding of gwl_logl_batch
(whose launch may split the bins differently); the rest of the output is left as it was; both
precisions, at tuned and heuristic shapes, and under graph capture with the length changed
between replays."""
import numpy as np
import pytest
import torch

from paper_1909_11873_amd import gwlike as gw
from paper_1909_11873_amd import synth
from tests.helpers import event_inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
TUNE = "paper_1909_11873_amd/tuning_gfx950.json"


def _event(cfg, f_hi=None):
    spec, f, psd, data, dets = event_inputs(cfg, f_hi=f_hi)
    t = lambda x: torch.tensor(x, device=DEV)
    return spec, gw.Event(t(data), t(psd), dets, t(f), spec.df)


@pytest.mark.parametrize("cfg,B,f_hi", [(1, 8192, None), (0, 1000, None), (1, 193, 300.0)])
def test_live_rows_equal_a_full_call(cfg, B, f_hi):
    gw.autotune_load(TUNE)
    spec, ev = _event(cfg, f_hi)
    th = torch.tensor(synth.theta_batch(spec, B), device=DEV)
    for prec in ("fp64", "mixed"):
        ref = gw.logl(th, ev, prec)
        full = gw.logl_live(th, torch.tensor(B, dtype=torch.int64, device=DEV), ev, prec)
        tol = 1e-9 * ref.abs().clamp(min=1.0) if prec == "fp64" else 2e-4
        assert bool(((full - ref).abs() <= tol).all()), prec
        for n in (0, 1, 63, 64, 65, B // 3, B - 1, B, B + 100):
            live = torch.tensor(n, dtype=torch.int64, device=DEV)
            out = torch.full((B,), 123.5, dtype=torch.float64, device=DEV)
            gw.logl_live(th, live, ev, prec, out=out)
            k = min(n, B)
            assert torch.equal(out[:k], full[:k]), (prec, n)
            assert bool((out[k:] == 123.5).all()), (prec, n)
    ev.close()


def test_live_length_changes_between_graph_replays():
    spec, ev = _event(1)
    B = 2048
    th = torch.tensor(synth.theta_batch(spec, B), device=DEV)
    live = torch.tensor(B, dtype=torch.int64, device=DEV)
    full = gw.logl_live(th, live, ev, "mixed")
    out = torch.zeros(B, dtype=torch.float64, device=DEV)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        gw.logl_live(th, live, ev, "mixed", out=out)           # reserves the workspace on s
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        gw.logl_live(th, live, ev, "mixed", out=out)
    for n in (B, 700, 0, 1, 1999):
        out.fill_(-7.0)
        live.fill_(n)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[:n], full[:n]) and bool((out[n:] == -7.0).all()), n
    ev.close()


def test_live_rejections():
    spec, ev = _event(0)
    th = torch.tensor(synth.theta_batch(spec, 10), device=DEV)
    with pytest.raises(ValueError):
        gw.logl_live(th, torch.tensor(3, dtype=torch.int32, device=DEV), ev)   # not int64
    L = gw.lib()
    import ctypes
    out = torch.empty(10, dtype=torch.float64, device=DEV)
    st = L.gwl_logl_batch_live(ev.handle, ctypes.c_void_p(th.data_ptr()), 10, None, gw.GWL_MIXED,
                               ctypes.c_void_p(out.data_ptr()), None)
    assert st == -1                                                         # live is required
    ev.close()
    cspec, f, psd, data, dets = event_inputs(0)
    t = lambda x: torch.tensor(x, device=DEV)
    cev = gw.Event(t(data), t(psd), dets, t(f), cspec.df, calibration_nodes=4)
    thc = torch.zeros(10, 11 + 8, dtype=torch.float64, device=DEV)
    with pytest.raises(gw.GWLError):
        gw.logl_live(thc, torch.tensor(3, dtype=torch.int64, device=DEV), cev)
    cev.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("cfg,B,f_hi,ndet", [(1, 700, 700.0, None), (1, 8192, 700.0, 2), (1, 300, 700.0, 1), (0, 1000, None, None),
                                             (1, 33000, 300.0, 4)])
def test_a_points_bits_are_its_own(cfg, B, f_hi, ndet, prec):
    """Whatever the rows past *live hold (other draws, points far away in time, NaN, infinities) and whichever
    points share its group of 64, a live point's value has the same bits: points of every level of rows and of
    none, in two orders, and NaN only where the point itself is outside the model's domain."""
    spec, f, psd, data, dets = event_inputs(cfg, f_hi=f_hi, ndet=ndet)
    t = lambda x: torch.tensor(x, device=DEV)
    ev = gw.Event(t(data), t(psd), dets, t(f), spec.df)
    th = np.tile(synth.theta_batch(spec, min(B, 4096)), (-(-B // 4096), 1))[:B]
    rng = np.random.default_rng(7)
    th[:, 0] = rng.uniform(1.0, 60.0, B)
    far = rng.random(B)
    th[:, 10] = np.where(far < 0.7, 0.1, np.where(far < 0.85, 0.28, 0.4 / spec.df)) * rng.uniform(-1.0, 1.0, B)
    th[17, 1] = 1.5
    live = B - 131
    n = torch.tensor(live, dtype=torch.int64, device=DEV)

    def call(rows):
        out = torch.full((B,), -3.0, dtype=torch.float64, device=DEV)
        gw.logl_live(t(rows), n, ev, prec, out=out)
        assert bool((out[live:] == -3.0).all())
        return out[:live].cpu().numpy()
    want = call(th)
    assert np.isnan(want).sum() == 1 and np.isnan(want[17])
    for column, value in ((slice(None), 0.0), (10, 1e3), (10, 1e300), (0, np.nan), (slice(None), np.inf)):
        rows = th.copy()
        rows[live:, column] = value
        assert np.array_equal(call(rows), want, equal_nan=True), (column, value)
    order = rng.permutation(live)
    rows = th.copy()
    rows[:live] = th[order]
    assert np.array_equal(call(rows), want[order], equal_nan=True)
    full = gw.logl(t(th), ev, prec).cpu().numpy()[:live]
    ok = np.isfinite(want)
    tol = 1e-9 * np.maximum(np.abs(full[ok]), 1.0) if prec == "fp64" else 1e-3
    assert (np.abs(want[ok] - full[ok]) <= tol).all()
    ev.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("B,f_hi", [(100, 700.0), (16384, 2048.0), (40000, 2048.0)])
def test_a_reserved_live_call_is_captured(B, f_hi, prec):
    """gwl_event_reserve for a value call of this size also covers the live-length call, whose launch has a shape
    of its own: captured with no call before it, it replays the eager call's values."""
    spec, ev = _event(1, f_hi)
    th = torch.tensor(np.tile(synth.theta_batch(spec, 100), (-(-B // 100), 1))[:B], device=DEV)
    live = torch.tensor(B - 3, dtype=torch.int64, device=DEV)
    out = torch.zeros(B, dtype=torch.float64, device=DEV)
    s = torch.cuda.Stream()
    gw.reserve(ev, B, prec, stream=s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        gw.logl_live(th, live, ev, prec, out=out)
    want = gw.logl_live(th, live, ev, prec)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[:B - 3], want[:B - 3]) and bool((out[B - 3:] == 0.0).all())
    ev.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nd,duration,f_hi,uniform", [(3, 8.0, 400.0, False), (1, 8.0, 700.0, False), (2, 64.0, 300.0, True),
                                                      (3, 128.0, 250.0, False)])
def test_live_calls_over_grids(nd, duration, f_hi, uniform, prec):
    """Levels on grids without a fixed step (no rotation of the phasors) and on long segments, where there are three:
    points of each and of none against the same bins with two neighbours swapped, which have no rows."""
    df = 1.0 / duration
    f = synth.freq_grid(20.0, f_hi, df)
    if not uniform:
        f = f + 0.2 * df * np.sin(np.arange(len(f)) * 1.7)
    psd = np.stack([synth.psd_fit(f)] * nd)
    dets = np.array([synth.detector_rad(n) for n in ("D1", "D2", "D3")[:nd]])
    data = np.stack([synth.noise(700 + i, psd[i], df) for i in range(nd)])
    k = len(f) // 2
    swap = np.r_[0:k, k + 1, k, k + 2:len(f)]
    mk = lambda i: gw.Event(torch.tensor(np.ascontiguousarray(data[:, i]), device=DEV),
                            torch.tensor(np.ascontiguousarray(psd[:, i]), device=DEV), dets,
                            torch.tensor(f[i], device=DEV), df)
    ev, plain = mk(np.arange(len(f))), mk(swap)
    rng = np.random.default_rng(17)
    th = synth.prior_draw(rng, 500)
    th[:, 0] = rng.uniform(1.0, 60.0, 500)
    th[:, 4] = 100.0
    kind = rng.integers(0, 4, 500)
    th[kind == 1, 10] = rng.uniform(-0.5, 0.5, (kind == 1).sum())
    th[kind == 2, 10] = rng.uniform(-0.4, 0.4, (kind == 2).sum()) * duration
    t = torch.tensor(th, device=DEV)
    n = torch.tensor(437, dtype=torch.int64, device=DEV)
    got = gw.logl_live(t, n, ev, prec)[:437].cpu().numpy()
    want = gw.logl(t, plain, prec)[:437].cpu().numpy()
    dn = np.sqrt(sum(float((4 * df * np.abs(d) ** 2 / s).sum()) for d, s in zip(data, psd)))
    hn = dn + np.sqrt(np.maximum(dn ** 2 - 2.0 * want, 0.0))
    tol = 1e-13 * hn * dn + 1e-9 if prec == "fp64" else 1e-3
    assert (np.abs(got - want) <= tol).all(), np.abs(got - want).max()
    ev.close()
    plain.close()
