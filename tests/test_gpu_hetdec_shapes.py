"""Matrix-core form of the time-domain front end at the edges of its splits:
the shortest filter it takes, each division of the taps over the waves, one
and two window buffers, windows past LDS (the direct sum), ragged ends and
series shorter than one block, and samples that are not finite.

Bar: every output is a sum of L products whose longest chain of roundings is
Kd / (2 WK) + WK + 3 additions (Kd = L + 7 D taps with the zero ones, WK >= 4
partial sums), then a phase factor good to a few ulp, so
|d| <= (Kd / 8 + 24) 2^-24 sum_i |h_i| max|x|."""
import numpy as np
import pytest

from oracle import heterodyne as oh

pytestmark = pytest.mark.gpu


def _bar(D, K, x):
    h = oh.kaiser_lowpass(D, K, 8.0)
    return ((len(h) + 7 * D) / 8 + 24) * 2.0 ** -24 * np.sum(np.abs(h)) * np.max(np.abs(x))


def _run(gpu_lib, x, dt, fh, D, K, n_out):
    import torch
    plan = gpu_lib.HetdecPlan(len(x), dt, fh, D, K, 8.0, n_out)
    out = plan.run(torch.from_numpy(x).cuda()).cpu().numpy()
    plan.close()
    return out


@pytest.mark.parametrize("D,K,n_out", [
    (2, 2, 700),        # the shortest filter of this form (9 taps)
    (2, 1, 200),        # 5 taps: the direct sum
    (3, 40, 1100),      # a window chunk shorter than two groups of taps
    (10, 8, 5), (10, 20, 3000),
    (25, 16, 129),      # one output past a block
    (50, 16, 128), (64, 20, 1000),
    (100, 16, 300), (128, 16, 260),   # two buffers, one buffer
    (250, 16, 70),      # window past LDS: the direct sum
])
def test_shapes_against_oracle(gpu_lib, D, K, n_out):
    rng = np.random.default_rng(100 * D + K)
    dt, fh = 1.0 / 512.0, 61.3
    n_raw = max(1, n_out * D - 3 * D // 2 + 1)
    x = rng.standard_normal(n_raw).astype(np.float32)
    ref = oh.heterodyne_decimate(x.astype(np.float64), dt, fh, D, K, 8.0, n_out)
    err = np.max(np.abs(_run(gpu_lib, x, dt, fh, D, K, n_out) - ref))
    print(f"hetdec D={D} K={K} n_out={n_out}: max|d| = {err:.2e}, bar {_bar(D, K, x):.2e}", flush=True)
    assert err <= _bar(D, K, x)


def test_many_blocks_per_workgroup(gpu_lib):
    """More blocks than workgroups take in one round, at the widest row tiles."""
    rng = np.random.default_rng(5)
    D, K, dt, fh, n_out = 10, 8, 1.0 / 512.0, 61.3, 700001
    x = rng.standard_normal(n_out * D).astype(np.float32)
    got = _run(gpu_lib, x, dt, fh, D, K, n_out)
    js = np.concatenate([np.arange(3), [511, 512, 513, 1023, 1024, n_out - 1], rng.integers(0, n_out, 300)])
    ref = oh.heterodyne_decimate_at(x, dt, fh, D, K, 8.0, js)
    assert np.max(np.abs(got[js] - ref)) <= _bar(D, K, x)


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
def test_non_finite_sample_stays_in_its_outputs(gpu_lib, value):
    """Only the outputs whose filter reaches the sample lose their value."""
    rng = np.random.default_rng(9)
    D, K, dt, fh, n_out, m = 20, 8, 1.0 / 512.0, 61.3, 1500, 11007
    x = rng.standard_normal(n_out * D).astype(np.float32)
    ref = oh.heterodyne_decimate(x.astype(np.float64), dt, fh, D, K, 8.0, n_out)
    bar = _bar(D, K, x)
    x[m] = value
    got = _run(gpu_lib, x, dt, fh, D, K, n_out)
    # outer taps of a Kaiser sinc are tiny but not zero, except at whole multiples of D
    reach = np.abs(np.arange(n_out) * D - m) <= K * D
    assert not np.any(np.isfinite(got[reach]))
    assert np.max(np.abs(got[~reach] - ref[~reach])) <= bar
