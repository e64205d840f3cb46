"""The FP64 outputs of the resampler (t_m, u, A', B', C') against the timing chain in
extended precision, at both sides of the limits between the interpolated and the
per-sample chain.

Bars: the inversion's residual of 1e-12 s and the rounding of T and t_b to FP64 (two
ulp of the series' length) for t_m, the same over dt for u; 2e-13 relative for
the antenna sums (the remainder 1e-13 allowed to a and b, and roundings)."""
import numpy as np
import pytest

from oracle import fstat as of
from paper_0912_4255_amd import synth
from paper_0912_4255_amd.synth import Binary
from tests.helpers import to_gpu

pytestmark = pytest.mark.gpu

LD = np.longdouble
TWO_PI = 8 * np.arctan(LD(1))


def _exact(w, al, de, orbit):
    """t_m and u by fixed point in extended precision."""
    e, det = w.eph, w.detectors[0]
    al, de = LD(al), LD(de)
    ts, dt = LD(w.segment.t_start), LD(w.segment.dt)
    tb = np.arange(w.segment.n).astype(LD) * dt
    target = tb
    if orbit:
        target = tb + LD(orbit.a_p) * np.sin(TWO_PI * ((ts + tb - LD(orbit.t_asc)) / LD(orbit.p_orb)))
    n = np.array([np.cos(de) * np.cos(al), np.cos(de) * np.sin(al), np.sin(de)])
    T = target
    for _ in range(12):
        tau = ts + T
        lam = LD(e.lambda0) + TWO_PI * tau / LD(e.p_orb)
        th = LD(e.theta0) + TWO_PI * tau / LD(e.p_sid) + LD(det.lon)
        ring, au, eps, lat = LD(e.re_c) * np.cos(LD(det.lat)), LD(e.au_c), LD(e.eps), LD(det.lat)
        r = (au * np.cos(lam) + ring * np.cos(th), au * np.cos(eps) * np.sin(lam) + ring * np.sin(th),
             au * np.sin(eps) * np.sin(lam) + LD(e.re_c) * np.sin(lat))
        T = target - (n[0] * r[0] + n[1] * r[1] + n[2] * r[2])
    return tb - T, T / dt


@pytest.mark.parametrize("n,dt,orbit", [
    (8000, 0.25, None), (8000, 0.94, None), (8000, 0.96, None), (8000, 2.0, None), (4000, 2.29, None), (3000, 4.0, None),
    (6000, 0.5, Binary(10.0, 14590.0, 1000.0)),      # near the limit of what an FFT's input takes
    (12000, 0.25, Binary(10.0, 7295.0, 1000.0)),
    (6000, 0.5, Binary(10.0, 30000.0, 1000.0)),      # near this one's
    (6000, 0.5, Binary(1.44, 68023.7, 2.3e4)),
    (6000, 2.0, Binary(1.44, 68023.7, 2.3e4)),
    (6000, 0.5, Binary(1.0, 3600.0, 9.0e4)),
])
def test_fp64_outputs(gpu_lib, n, dt, orbit):
    import torch
    w = synth.small_workload(n=n, dt=dt, taps=16, nfft_policy=synth.NFFT_SMOOTH7)
    rng = np.random.default_rng(n)
    x = (rng.standard_normal(n) + 1j * rng.standard_normal(n)).astype(np.complex64)
    gaps = np.array([[100, 300]], dtype=np.int64)
    plan = gpu_lib.Plan(w)
    row = [1.2, 0.3]
    if orbit:
        plan.set_binary(True)
        row += [orbit.a_p, orbit.p_orb, orbit.t_asc]
    tx, tg = to_gpu([x], [gaps])
    o = {k: v[0].cpu().numpy() for k, v in
         plan.resample(tx, tg, torch.tensor([row], dtype=torch.float64).cuda())[0].items()}
    plan.close()
    tm, u = _exact(w, row[0], row[1], orbit)
    bar = 1e-12 + 2 * np.spacing(n * dt)
    err_t, err_u = np.max(np.abs(o["tm"] - tm)), np.max(np.abs(o["u"] - u))
    ref = of.resample(x, gaps, w.segment, row[0], row[1], w.eph, w.detectors[0], w.kernel, w.taps, binary=orbit)
    m, a, b = ref["mask"], ref["a"], ref["b"]
    err_s = np.max(np.abs(o["abc"] / [np.sum(m * a * a), np.sum(m * b * b), np.sum(m * a * b)] - 1))
    print(f"n={n} dt={dt} {orbit}: t_m {float(err_t):.1e} s, u {float(err_u):.1e}, sums {err_s:.1e}", flush=True)
    assert err_t <= bar and err_u <= bar / dt + 2 * np.spacing(float(n)) and err_s <= 2e-13
