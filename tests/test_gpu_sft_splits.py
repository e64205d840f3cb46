"""SFT front end on the GPU at the edges of its kernels' splits, against the
FP64 oracle: grids on both sides of one DFT thread per root (M' up to and
above 256), bands stored short of the Dirichlet terms' reach (also by whole
workgroups of the merge), term counts with and without an instance of their
own, transform lengths past the 256-thread rows and columns passes, sets with
and without gaps.

Bar, as for the front end's other tests: max|d| <= 1e-4 max|x_oracle| (FP32
sums of at most M (2 dk + 1) terms and two FFT passes), gaps identical.
Inputs: seeded white-noise SFT bands of unit power, no normalisation."""
import numpy as np
import pytest

from oracle import sft as osft
from paper_0912_4255_amd import synth

pytestmark = pytest.mark.gpu


def _run(gpu_lib, slots, n_slots, band_bins, dk, low=0, high=0, edge_taper_s=2.0, T=8.0, f_bins=960):
    """Band of band_bins bins stored with its dk margin, less low and high
    bins at its ends."""
    import torch
    rng = np.random.default_rng(1000 * dk + len(slots) + 7 * low + high)
    k_lo = f_bins - band_bins // 2 - dk - 1 + low
    K = band_bins + 2 * (dk + 1) - low - high
    X = synth.sft_noise(rng, len(slots), K, 1.0).astype(np.complex64)
    band = band_bins / T
    ss = synth.SftSet(sft_len=4 * band_bins, dt_raw=T / (4 * band_bins), k_lo=k_lo, n_bins=K,
                      t_sft=np.array(slots, dtype=np.float64) * T, t_start=0.0, f_het=f_bins / T, band=band,
                      n_out=n_slots * band_bins, dk=dk, median_window=0, band_taper=0.05, edge_taper_s=edge_taper_s)
    ref, gref = osft.heterodyne_from_sfts(X.astype(np.complex128), ss.t_sft, ss.t_sft_len, ss.k_lo, ss.t_start,
                                          ss.f_het, ss.band, ss.n_out, dk=dk, median_window=1,
                                          band_taper=ss.band_taper, edge_taper_s=edge_taper_s, normalise_sfts=False)
    plan = gpu_lib.SftPlan(ss)
    out = torch.full((ss.n_out,), complex("nan"), dtype=torch.complex64, device="cuda")
    got = plan.heterodyne(torch.from_numpy(X).cuda(), out=out).cpu().numpy()
    gaps = plan.gaps
    plan.close()
    assert np.array_equal(gaps, gref)
    err, scale = np.max(np.abs(got - ref)), np.max(np.abs(ref))
    print(f"M = {len(slots)}, {band_bins} bins, dk = {dk}, cut {low}/{high}: {err / scale:.2e}", flush=True)
    assert err <= 1e-4 * scale
    for a, b in gaps:
        assert np.all(got[a:b] == 0)


@pytest.mark.parametrize("dk", [1, 2, 8, 16])
@pytest.mark.parametrize("low,high", [(0, 0), (1, 0), (3, 21), (25, 2)])
@pytest.mark.parametrize("M", [1, 7, 130])
def test_band_short_of_the_terms(gpu_lib, M, low, high, dk):
    _run(gpu_lib, list(range(M)), M, 32, dk, low, high)


@pytest.mark.parametrize("M", [255, 256, 257, 300])
@pytest.mark.parametrize("cut", [0, 12])
def test_grids_about_one_thread_per_root(gpu_lib, M, cut):
    _run(gpu_lib, list(range(M)), M, 32, 2, cut, cut)


@pytest.mark.parametrize("slots,n_slots", [([0, 2], 3), ([1, 2, 5], 8), (list(range(9)), 9)])
def test_gaps(gpu_lib, slots, n_slots):
    _run(gpu_lib, slots, n_slots, 4096, 4, f_bins=8000)


def _merge_by_fft(Xh, k_lo, M_grid, b_values, dk, kernel=None):
    """osft.merge_chunk of consecutive bins with the sum over the SFTs as one
    FFT per stored bin (the oracle takes a minute at 2^20 bins)."""
    K = Xh.shape[1]
    Y = np.fft.fft(Xh, n=M_grid, axis=0)  # [r][k]
    ks, r = b_values // M_grid, b_values % M_grid
    out = np.zeros(len(b_values), dtype=np.complex128)
    for d in range(-dk, dk + 1):
        k = ks + d
        ok = (k >= k_lo) & (k < k_lo + K)
        P = osft.dirichlet_large_n(b_values, k, M_grid)
        out[ok] += P[ok] * Y[r[ok], k[ok] - k_lo]
    return out


@pytest.mark.parametrize("M,band_bins", [
    (8, 131072),   # 2^20 points: rows of 4096
    (8, 262144),   # 2^21 points: rows of 4096, columns of 512
])
def test_lengths_past_the_small_workgroups(gpu_lib, monkeypatch, M, band_bins):
    rng = np.random.default_rng(M)
    X = rng.standard_normal((3, 40)) + 1j * rng.standard_normal((3, 40))
    b = np.arange(4 * 100, 4 * 140)
    assert np.allclose(_merge_by_fft(X, 100, 4, b, 2), osft.merge_chunk(X, 100, 4, b, 2), rtol=0, atol=1e-12)
    monkeypatch.setattr(osft, "merge_chunk", _merge_by_fft)
    _run(gpu_lib, list(range(M)), M, band_bins, 2, T=8192.0, f_bins=204800)
