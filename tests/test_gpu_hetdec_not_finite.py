"""Raw samples that are not finite in the matrix-core form of the time-domain
front end: stretches, single samples, infinities and overflows lose the outputs
whose filter reaches them and no other, and a stretch costs little time."""
import numpy as np
import pytest

from oracle import heterodyne as oh

pytestmark = pytest.mark.gpu

DT, FH = 1.0 / 512.0, 61.3
SHAPES = [(2, 2, 700), (10, 8, 9000), (25, 16, 3000), (64, 8, 1500), (64, 16, 1500), (100, 16, 600), (128, 16, 600)]


def _run(gpu_lib, x, D, K, n_out):
    import torch
    plan = gpu_lib.HetdecPlan(len(x), DT, FH, D, K, 8.0, n_out)
    out = plan.run(torch.from_numpy(x).cuda()).cpu().numpy()
    plan.close()
    return out


def _clean(x, D, K, n_out, bad):
    """The oracle's series with the bad samples zeroed, which outputs reach one,
    and 2^-24 (Kd / 8 + 24) sum|h| max|x|, the bound on a sum's roundings (Kd = L + 7 D
    products in chains of at most Kd / 8)."""
    y = np.where(bad, 0.0, x).astype(np.float64)
    j = np.arange(n_out) * D
    c = np.concatenate([[0], np.cumsum(bad)])
    hi = np.minimum(j + K * D + 1, len(x))
    reach = c[hi] - c[np.minimum(np.maximum(j - K * D, 0), hi)] > 0
    h = oh.kaiser_lowpass(D, K, 8.0)
    bar = ((len(h) + 7 * D) / 8 + 24) * 2.0 ** -24 * np.sum(np.abs(h)) * np.max(np.abs(y))
    return oh.heterodyne_decimate_at(y, DT, FH, D, K, 8.0, np.flatnonzero(~reach)), reach, bar


@pytest.mark.parametrize("D,K,n_out", SHAPES)
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_stretch_and_single_samples(gpu_lib, D, K, n_out, value):
    """A stretch over several blocks, single samples at the series' ends and
    near the stretch, all at odd places."""
    rng = np.random.default_rng(D + K)
    n = n_out * D
    x = rng.standard_normal(n).astype(np.float32)
    bad = np.zeros(n, dtype=bool)
    bad[n // 3:n // 3 + n // 4 + 1] = True
    bad[[0, 3 * D + 1, n // 3 - 3 * K * D - 5, 11 * n // 12, n - 1]] = True
    x[bad] = value
    ref, reach, bar = _clean(x, D, K, n_out, bad)
    got = _run(gpu_lib, x, D, K, n_out)
    assert not np.any(np.isfinite(got[reach].real) & np.isfinite(got[reach].imag))
    if np.isnan(value):
        assert np.all(np.isnan(got[reach].real) & np.isnan(got[reach].imag))
    assert np.max(np.abs(got[~reach] - ref)) <= bar


def test_infinity_and_overflow_as_a_plain_sum(gpu_lib):
    """One infinity, and finite samples whose sum overflows: what the plain sum of
    the filter gives in FP32, infinite or NaN."""
    D, K, n_out = 20, 8, 800
    x = np.ones(n_out * D, dtype=np.float32)
    x[4007] = np.inf
    x[9000:9400] = 3e38
    h = oh.kaiser_lowpass(D, K, 8.0)
    got = _run(gpu_lib, x, D, K, n_out)
    j = np.arange(n_out) * D
    assert not np.any(np.isfinite(got[np.abs(j - 4007) <= K * D]))
    far = (np.abs(j - 4007) > K * D) & (np.abs(j - 9200) > K * D + 200)
    ref = oh.heterodyne_decimate(np.ones(n_out * D), DT, FH, D, K, 8.0, n_out)
    bar = ((len(h) + 7 * D) / 8 + 24) * 2.0 ** -24 * np.sum(np.abs(h))
    assert np.max(np.abs(got[far] - ref[far])) <= bar


def test_stretch_costs_little(gpu_lib):
    """An hour of NaN in ten days at 256 Hz lies in one or two workgroups, for
    which the whole call waits: at most twice the time of finite samples (it was 39
    times with every affected output summed by one thread)."""
    import torch
    D, K, n_out = 64, 16, 3456000
    x = torch.randn(n_out * D, device="cuda")
    out = torch.empty(n_out, dtype=torch.complex64, device="cuda")
    plan = gpu_lib.HetdecPlan(n_out * D, 1.0 / 256.0, FH, D, K, 8.0, n_out)

    def time():
        plan.run(x, out=out)
        ms = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            plan.run(x, out=out)
            b.record()
            b.synchronize()
            ms.append(a.elapsed_time(b))
        return min(ms)

    finite = time()
    x[50_000_000:50_000_000 + 3600 * 256] = float("nan")
    hour = time()
    plan.close()
    print(f"finite {1e3 * finite:.0f} us, an hour of NaN {1e3 * hour:.0f} us", flush=True)
    assert hour <= 2 * finite
