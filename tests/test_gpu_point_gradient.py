"""2F and its gradient with the interpolated timing chain against 64-bit automatic
differentiation, each component to FP32 rounding.

Bar: the weights, phases and products of a sample are good to about 8 roundings of
2^-24 and the terms add at random, as the gradient's own do, so its components,
over the candidates of a call, are off by 5e-7 of their norm; four times that is
allowed, 2e-6 (2F likewise).  For alpha and delta the constant part of the delay's
derivative D turns F_a and F_b as a whole, which leaves 2F as it is: what is left of
those terms is smaller by rms(D) / std(D), by which the bar is larger.  At the
fastest orbit that is interpolated, leaving out the slope of the heterodyne
correction's derivative over the window is seen."""
import math

import numpy as np
import pytest
import torch

from paper_0912_4255_amd import synth
from perf import cases as pc

BAR = 2e-6


def _problem(n, dt, dets, taps, order, orbit, kernel=synth.KERNEL_DIRICHLET, cands=6):
    w = synth.small_workload(n=n, dt=dt, kernel=kernel, taps=taps, n_det=dets, t_start=3.0e5, nfft_policy=synth.NFFT_SMOOTH7)
    rng = np.random.default_rng(n + order)
    xs, gaps = [], []
    for det in w.detectors:
        x = rng.standard_normal((n, 2)) @ [1, 1j] * math.sqrt(det.sigma2 / 2)
        x[n // 5:n // 5 + 300] = 0
        xs.append(torch.from_numpy(x.astype(np.complex64)))
        gaps.append(torch.tensor([[n // 5, n // 5 + 300]], dtype=torch.int64))
    cols = [100.0 + rng.uniform(-0.2, 0.2, cands) / dt, rng.uniform(-1e-9, 0.0, cands)]
    cols += [rng.uniform(-1, 1, cands) * s for s in (1e-15, 1e-21)[:order - 1]] + list(synth.uniform_sky(rng, cands).T)
    if orbit:
        cols += [np.full(cands, orbit[0]), orbit[1] * (1 + 1e-3 * np.arange(cands)), rng.uniform(0, orbit[1], cands)]
    return w, xs, gaps, torch.from_numpy(np.column_stack(cols))


def _exact(w, xs, gaps, theta, order, resampled=pc._resampled):
    F, G = [], []
    t = torch.arange(w.segment.n, dtype=torch.float64, device=theta.device) * w.segment.dt
    for row in theta:
        th = row.clone().requires_grad_()
        sky = th[1 + order:]
        rs = [resampled(w, k, x, g, sky[0], sky[1], sky[2:] if len(sky) > 2 else None) for k, (x, g) in enumerate(zip(xs, gaps))]
        ya, yb = pc._integrands(w, rs, th[1:1 + order])
        cyc = (th[0] - w.segment.f_het) * t
        e = torch.exp(-2j * math.pi * (cyc - torch.floor(cyc.detach())))
        twoF = pc._twoF((ya * e).sum(), (yb * e).sum(), pc._sums(w, rs))
        G.append(torch.autograd.grad(twoF, th)[0])
        F.append(twoF.detach())
    return torch.stack(F), torch.stack(G)


def _bars(w, theta, order):
    """Per component: BAR, for alpha and delta times rms(D) / std(D)."""
    bars = np.full(theta.shape[1], BAR)
    t = w.segment.t_start + torch.arange(w.segment.n, dtype=torch.float64) * w.segment.dt
    sky = theta[:, 1 + order:3 + order].cpu()
    for i in range(2):
        step = 1e-4 * torch.eye(2, dtype=torch.float64)[i]
        D = torch.stack([(pc._roemer(t, *(s + step), w.eph, w.detectors[0])[0] - pc._roemer(t, *(s - step), w.eph, w.detectors[0])[0])
                         / 2e-4 for s in sky])
        bars[1 + order + i] *= float((D.square().mean(dim=1).sqrt() / D.std(dim=1)).max())
    return bars


FASTEST = (0.05, 13200.0)  # 2 pi 146 dt / P_b = 0.0347 at dt = 0.5 s, where 0.035 is the limit


@pytest.mark.gpu
@pytest.mark.parametrize("n,dt,dets,taps,order,orbit,kernel", [
    (30000, 0.5, 1, 16, 1, FASTEST, synth.KERNEL_DIRICHLET),
    (100000, 0.5, 1, 16, 1, FASTEST, synth.KERNEL_DIRICHLET),   # weights without their small-angle factor
    (30001, 0.5, 2, 8, 2, FASTEST, synth.KERNEL_LANCZOS),
    (40000, 1.0, 1, 24, 3, (1.44, 68023.7), synth.KERNEL_DIRICHLET),
    (30000, 0.5, 1, 16, 1, (1.0, 3600.0), synth.KERNEL_DIRICHLET),   # every sample's chain
    (30000, 0.5, 1, 16, 1, None, synth.KERNEL_DIRICHLET),
    (200000, 1.0, 2, 16, 2, None, synth.KERNEL_DIRICHLET),
    (9000, 4.3, 1, 16, 3, None, synth.KERNEL_DIRICHLET),
    (9000, 5.0, 1, 16, 1, None, synth.KERNEL_LANCZOS),               # every sample's chain
])
def test_components(gpu_lib, n, dt, dets, taps, order, orbit, kernel):
    w, xs, gaps, theta = _problem(n, dt, dets, taps, order, orbit, kernel)
    xs, gaps, theta = [x.cuda() for x in xs], [g.cuda() for g in gaps], theta.cuda()
    w.gaps = [g.cpu().numpy() for g in gaps]
    plan = gpu_lib.Plan(w)
    plan.set_spin_order(order)
    plan.set_binary(orbit is not None)
    F, g = plan.backward(xs, gaps, theta, torch.ones(len(theta), dtype=torch.float32, device="cuda"))
    F0 = plan.point(xs, gaps, theta)
    plan.close()
    rF, rg = _exact(w, xs, gaps, theta, order)
    err = ((g - rg).norm(dim=0) / rg.norm(dim=0)).cpu().numpy()
    print(f"n={n} dt={dt} {orbit}: 2F {float((F - rF).norm() / rF.norm()):.1e}, gradient "
          + " ".join(f"{v:.1e}" for v in err), flush=True)
    assert float((F - rF).norm() / rF.norm()) <= BAR and float((F0 - rF).norm() / rF.norm()) <= BAR
    assert np.all(err <= _bars(w, theta, order))


def _flat_correction(w, i, x, gaps, alpha, delta, orbit):
    """pc._resampled with the heterodyne correction's derivative taken at the
    output's position for all taps of its window."""
    z, a, b, T, d, m = pc._resampled(w, i, x, gaps, alpha, delta, orbit)
    seg, eph, det = w.segment, w.eph, w.detectors[i]
    at = T.detach()
    D = pc._roemer(seg.t_start + at, alpha, delta, eph, det)[0]
    D = D - pc._orbit(pc._solve(seg.t_start + at + D, lambda t: pc._orbit(t, orbit)), orbit)[0]
    fixed = dict(alpha=alpha.detach(), delta=delta.detach(), orbit=orbit.detach())
    # the series with the correction frozen still moves with T: interpolate it at the moving position
    t = torch.arange(seg.n, dtype=torch.float64) * seg.dt
    tm = pc._roemer(seg.t_start + t, fixed["alpha"], fixed["delta"], eph, det)[0]
    dk = tm - pc._orbit(pc._solve(seg.t_start + t + tm, lambda s: pc._orbit(s, fixed["orbit"])), fixed["orbit"])[0]
    zk = x.to(torch.complex128) * torch.exp(-2j * math.pi * (seg.f_het * dk))
    u = T / seg.dt
    j = torch.floor(u.detach())
    frac, j = u - j, j.long()
    out = 0.0
    for k in range(1, w.taps + 1):
        pos = j - w.taps // 2 + k
        tap = torch.where((pos >= 0) & (pos < seg.n), zk[pos.clamp(0, seg.n - 1)], torch.zeros((), dtype=zk.dtype))
        out = out + pc._weight(frac + (w.taps / 2 - k), w.kernel, w.taps, seg.n) * tap
    return out * torch.exp(-2j * math.pi * seg.f_het * (D - D.detach())), a, b, T, d, m


def test_bar_sees_the_slope_of_the_correction():
    """On the CPU: the gradient without that slope is off by ten times the bar and
    more in the orbit's components."""
    w, xs, gaps, theta = _problem(30000, 0.5, 1, 16, 1, FASTEST, cands=3)
    _, g = _exact(w, xs, gaps, theta, 1)
    _, flat = _exact(w, xs, gaps, theta, 1, resampled=_flat_correction)
    err = ((flat - g).norm(dim=0) / g.norm(dim=0)).numpy()
    print(" ".join(f"{v:.1e}" for v in err))
    assert np.all(err[4:] >= 10 * _bars(w, theta, 1)[4:]) and np.max(err) <= 1e-2
