"""The resampler with the interpolated timing chain (runs of 128 samples) at the
edges of its tiles and of the range it takes, against the oracle, with the bars
of the resampling parity test: |dz~| <= 3e-6 rms, |da|, |db| <= 1e-6,
|dt_m| <= 1e-9 s, the SSB mask bit for bit, A', B', C' to 1e-10."""
import numpy as np
import pytest

from oracle import fstat as of
from paper_0912_4255_amd import synth
from paper_0912_4255_amd.synth import Binary
from tests.helpers import make_inputs, to_gpu

pytestmark = pytest.mark.gpu


def _check(gpu_lib, w, xs, gaps, skies, orbits=None):
    import torch
    plan = gpu_lib.Plan(w)
    rows = np.array(skies, dtype=np.float64)
    if orbits is not None:
        plan.set_binary(True)
        rows = np.column_stack([rows, [[o.a_p, o.p_orb, o.t_asc] for o in orbits]])
    tx, tg = to_gpu(xs, gaps)
    out = plan.resample(tx, tg, torch.from_numpy(np.ascontiguousarray(rows)).cuda())
    n = w.segment.n
    for X, det in enumerate(w.detectors):
        for s, (al, de) in enumerate(skies):
            ref = of.resample(xs[X], gaps[X], w.segment, al, de, w.eph, det, w.kernel, w.taps,
                              binary=orbits[s] if orbits is not None else None)
            o = {k: v[s].cpu().numpy() for k, v in out[X].items()}
            assert np.max(np.abs(o["tm"] - ref["tm"])) < 1e-9
            assert np.max(np.abs(o["a"] - ref["a"])) < 1e-6 and np.max(np.abs(o["b"] - ref["b"])) < 1e-6
            assert np.max(np.abs(o["u"] - ref["u"])) < 1e-9 / w.segment.dt
            rms = np.sqrt(np.mean(np.abs(ref["z"]) ** 2))
            assert np.max(np.abs(o["z"] - ref["z"])) <= 3e-6 * rms  # a delay past the segment: all zero
            bits = np.unpackbits(o["mask"].view(np.uint8), bitorder="little")
            assert np.array_equal(bits[:n].astype(bool), ref["mask"] > 0) and not bits[n:].any()
            m, a, b = ref["mask"], ref["a"], ref["b"]
            assert np.allclose(o["abc"], [np.sum(m * a * a), np.sum(m * b * b), np.sum(m * a * b)], rtol=1e-10, atol=0)
    plan.close()


@pytest.mark.parametrize("n,dt,n_det,kernel,taps", [
    (100, 4.0, 1, synth.KERNEL_DIRICHLET, 16),     # less than a run, every sample's chain
    (100, 2.0, 1, synth.KERNEL_DIRICHLET, 16),     # less than a run, interpolated
    (2048, 1.0, 1, synth.KERNEL_DIRICHLET, 16),    # one full tile
    (2049, 1.0, 2, synth.KERNEL_DIRICHLET, 2),     # one sample past it, odd length
    (33333, 0.25, 1, synth.KERNEL_DIRICHLET, 32),  # a flat kernel, the widest window
    (40000, 0.5, 2, synth.KERNEL_LANCZOS, 8),
    (6000, 2.3, 1, synth.KERNEL_DIRICHLET, 24),    # near the longest sampling interval interpolated
    (6000, 7.5, 1, synth.KERNEL_DIRICHLET, 24),    # past it
    (6000, 9.0, 1, synth.KERNEL_DIRICHLET, 24),
])
def test_tiles_against_oracle(gpu_lib, n, dt, n_det, kernel, taps):
    w = synth.small_workload(n=n, dt=dt, kernel=kernel, taps=taps, n_det=n_det, t_start=2.0e5,
                             nfft_policy=synth.NFFT_SMOOTH7)
    if n > 5000:  # gaps over whole runs, on run edges, of one sample, and at both ends
        g = [[0, 130], [256, 384], [1000, 1001], [1100, 2300], [2432, 2433], [n - 7, n]]
        w.gaps = [np.array(g, dtype=np.int64) for _ in w.detectors]
    xs, gaps = make_inputs(w, seed=n)
    _check(gpu_lib, w, xs, gaps, [(1.2, 0.3), (4.1, -0.8)])


def test_orbits_share_a_call(gpu_lib):
    """Slow orbits (interpolated) and fast ones (every sample) in one call."""
    w = synth.small_workload(n=30001, dt=0.5, taps=16, t_start=1.0e5, nfft_policy=synth.NFFT_SMOOTH7)
    w.gaps = [np.array([[700, 900], [5000, 9000]], dtype=np.int64)]
    xs, gaps = make_inputs(w, seed=3)
    _check(gpu_lib, w, xs, gaps, [(1.2, 0.3), (4.1, -0.8), (2.0, 1.0)],
           [Binary(1.44, 68023.7, 2.3e4), Binary(1.0, 3600.0, 9.0e4), Binary(0.0, 5.0e4, 0.0)])
