"""The point 2F and its adjoint with the interpolated timing chain (runs of 256
samples) at the edges of its splits, against the oracle.

Bars as in the other point tests: |d2F| <= 1e-4 max(2F, 4); the gradient, each
component scaled by (1/T0, 1/T0^2, ..., 1e-5, 1e-5[, 1e-3, 1, 10]), within 1e-3
of max(largest scaled component, 1) of the oracle's (2e-3 for the orbit)."""
import numpy as np
import pytest

from oracle import fstat as of  # noqa: F401
from oracle import grad as og
from paper_0912_4255_amd import synth
from tests.helpers import make_inputs, to_gpu

pytestmark = pytest.mark.gpu


def _case(n, dt, n_det=1, kernel=synth.KERNEL_DIRICHLET, taps=16, seed=1, gaps=()):
    w = synth.small_workload(n=n, dt=dt, kernel=kernel, taps=taps, n_det=n_det, t_start=3.0e5,
                             nfft_policy=synth.NFFT_SMOOTH7)
    w.gaps = [np.array(gaps, dtype=np.int64).reshape(-1, 2) for _ in w.detectors]
    xs, gs = make_inputs(w, seed=seed)
    return w, xs, gs


def _theta(w, order, seed, n=2):
    rng = np.random.default_rng(seed)
    B = 1.0 / w.segment.dt
    sky = synth.uniform_sky(rng, n)
    cols = [100.0 + rng.uniform(-0.2, 0.2, n) * B, rng.uniform(-1e-9, 0.0, n)]
    cols += [rng.uniform(-1, 1, n) * s for s in (1e-15, 1e-21)[:order - 1]]
    return np.column_stack(cols + [sky])


def _check(gpu_lib, w, xs, gaps, th, order, binary=False):
    import torch
    plan = gpu_lib.Plan(w)
    plan.set_spin_order(order)
    plan.set_binary(binary)
    tx, tg = to_gpu(xs, gaps)
    t = torch.from_numpy(np.ascontiguousarray(th)).cuda()
    F = plan.point(tx, tg, t).cpu().numpy()
    F2, g = plan.backward(tx, tg, t, torch.ones(len(th), dtype=torch.float32).cuda())
    F2, g = F2.cpu().numpy(), g.cpu().numpy()
    plan.close()
    prob = og.PointProblem(xs, gaps, w.segment, list(w.detectors), w.eph, w.kernel, w.taps, binary=binary)
    T0 = w.segment.n * w.segment.dt
    main = np.array([T0 ** -(j + 1) for j in range(order + 1)] + [1e-5, 1e-5])
    orb = np.array([1e-3, 1.0, 10.0])
    for i, row in enumerate(th):
        ref = prob.twoF(row)
        assert abs(F[i] - ref) <= 1e-4 * max(ref, 4.0) and abs(F2[i] - ref) <= 1e-4 * max(ref, 4.0), (i, F[i], F2[i], ref)
        rg = og.gradient(prob, row)
        k = len(main)
        a, b = g[i, :k] * main, rg[:k] * main
        assert np.all(np.abs(a - b) <= 1e-3 * max(np.max(np.abs(b)), 1.0)), (i, a, b)
        if binary:
            a, b = g[i, k:] * orb, rg[k:] * orb
            assert np.all(np.abs(a - b) <= 2e-3 * max(np.max(np.abs(b)), 1.0)), (i, a, b)


@pytest.mark.parametrize("n,dt,n_det,order,kernel,taps", [
    (130, 4.0, 1, 1, synth.KERNEL_DIRICHLET, 16),      # less than a run
    (32768, 0.5, 1, 1, synth.KERNEL_DIRICHLET, 16),    # the longest series with one row per wave
    (32769, 0.5, 2, 2, synth.KERNEL_DIRICHLET, 24),    # the shortest with a run per wave, odd length, one-sample row
    (33001, 0.25, 1, 3, synth.KERNEL_LANCZOS, 8),      # last run partial
    (40000, 2.0, 1, 1, synth.KERNEL_DIRICHLET, 2),
    (40001, 1.0, 2, 1, synth.KERNEL_DIRICHLET, 32),    # widest window
    (262145, 0.5, 1, 1, synth.KERNEL_DIRICHLET, 16),   # two runs per wave
    (5000, 4.2, 1, 1, synth.KERNEL_DIRICHLET, 16),     # near the longest sampling interval interpolated
    (5000, 5.0, 2, 1, synth.KERNEL_DIRICHLET, 16),     # past it: the chain of every sample
])
def test_splits_against_oracle(gpu_lib, n, dt, n_det, order, kernel, taps):
    w, xs, gaps = _case(n, dt, n_det, kernel, taps)
    _check(gpu_lib, w, xs, gaps, _theta(w, order, n, 1 if n > 50000 else 2), order)


def test_gaps_at_run_edges(gpu_lib):
    """Gaps that cover whole runs, end on run edges, lie inside one row, and reach both ends."""
    w, xs, gaps = _case(9000, 2.0, 2, gaps=[(0, 300), (512, 768), (1000, 1024), (1600, 1601), (2048, 4100), (8990, 9000)])
    _check(gpu_lib, w, xs, gaps, _theta(w, 1, 4, 2), 1)


def test_orbits_share_a_call(gpu_lib):
    """Slow orbits (interpolated), fast ones (every sample) and refused ones in one call."""
    import torch
    w, xs, gaps = _case(30000, 0.5, gaps=[(700, 900)])
    orbits = np.array([[1.5, 90000.0, 1.0e5], [1.44, 7200.0, 3.0e5], [0.0, 50000.0, 0.0]])
    th = np.column_stack([_theta(w, 1, 8, 3), orbits])
    _check(gpu_lib, w, xs, gaps, th, 1, binary=True)
    plan = gpu_lib.Plan(w)
    plan.set_binary(True)
    tx, tg = to_gpu(xs, gaps)
    bad = np.vstack([th, th[0]])
    bad[3, 4] = 150.0
    F = plan.point(tx, tg, torch.from_numpy(bad).cuda()).cpu().numpy()
    assert np.all(np.isfinite(F[:3])) and np.isnan(F[3])
    plan.close()


def test_workspace_of_the_coarsest_split_is_enough(gpu_lib):
    """A workspace that holds one partial sum per 128 rows and candidate is
    accepted, and a large call is cut into launches without changing a bit."""
    import torch
    w, xs, gaps = _case(20000, 2.0)
    plan = gpu_lib.Plan(w)
    tx, tg = to_gpu(xs, gaps)
    th = _theta(w, 1, 3, 400)
    t = torch.from_numpy(th).cuda()
    g1 = torch.ones(400, dtype=torch.float32).cuda()
    F, g = plan.backward(tx, tg, t, g1)
    Fs, gs = plan.backward(tx, tg, t[:3].contiguous(), g1[:3].contiguous())
    assert torch.equal(F[:3], Fs) and torch.equal(g[:3], gs)
    rows = -(-20000 // 64)
    small = torch.empty(256 + 2 * -(-rows // 128) * 512, dtype=torch.uint8, device="cuda")
    Fc, gc = plan.backward(tx, tg, t[:2].contiguous(), g1[:2].contiguous(), ws=small)
    assert torch.allclose(Fc, F[:2], rtol=1e-6) and torch.allclose(gc, g[:2], rtol=1e-6, atol=0)
    with pytest.raises(gpu_lib.RsfError):
        plan.backward(tx, tg, t[:2].contiguous(), g1[:2].contiguous(), ws=small[:-512].contiguous())
    plan.close()
