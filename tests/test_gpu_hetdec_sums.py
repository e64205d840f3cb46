"""The sums of the time-domain front end, tap by tap and to FP32 rounding: every
tap has its place and value, an output's bits depend on the filter and not on the
length of the series, and the error against 64 bits is that of a sum in
short chains."""
import numpy as np
import pytest

from oracle import heterodyne as oh

pytestmark = pytest.mark.gpu

DT, FH = 1.0 / 512.0, 61.3
# 4, 8 and 16 waves along the taps, one and two window buffers, an odd D, groups of taps
# past the filter's end, and the direct sum (D = 128, K = 20; D = 137, K = 2; D = 250; K = 1)
SHAPES = [(2, 2), (3, 40), (10, 8), (10, 20), (25, 12), (25, 16), (32, 16), (50, 16), (64, 8), (64, 12), (64, 16),
          (64, 20), (100, 16), (120, 3), (128, 16), (100, 20), (128, 20), (137, 2), (250, 8), (16, 1)]


def _run(gpu_lib, x, D, K, n_out):
    import torch
    x = x if torch.is_tensor(x) else torch.from_numpy(x).cuda()
    plan = gpu_lib.HetdecPlan(x.numel(), DT, FH, D, K, 8.0, n_out)
    out = plan.run(x)
    plan.close()
    return out


def _taps(D, K):
    """g[i] = h[i] exp(-2 pi i f (c - i) dt) in FP64."""
    h = oh.kaiser_lowpass(D, K, 8.0)
    cyc = FH * DT * (K * D - np.arange(len(h)))
    return h * np.exp(-2j * np.pi * (cyc - np.rint(cyc)))


@pytest.mark.parametrize("n_out", [0, 300000])
@pytest.mark.parametrize("D,K", SHAPES)
def test_every_tap(gpu_lib, D, K, n_out):
    """Unit impulses far enough apart that an output reaches one at most, one for
    each residue of the sample index mod D, so that each tap is met alone, in a
    series of that length and in one long enough for the widest row tiles.  The
    output is the tap, rounded to FP32 (2^-24 |g|), times a phase whose angle is
    rounded to FP32 below half a turn (2^-25 turns: 3.2 x 2^-24) and whose sine and
    cosine are good to 2 ulp, with three more roundings: at most 9 x 2^-24 |g|."""
    L = 2 * K * D + 1
    step = (L // D + 2) * D + 1               # every residue once
    n_out = max(n_out, (step * D) // D + 2 * K + 2)
    x = np.zeros(n_out * D, dtype=np.float32)
    m = K * D + step * np.arange(D)
    x[m] = 1.0
    got = _run(gpu_lib, x, D, K, n_out).cpu().numpy().astype(np.complex128)
    ref = np.zeros(n_out, dtype=np.complex128)
    g = _taps(D, K)
    met = np.zeros(L, dtype=int)
    for mm in m:
        j = np.arange(-(-(mm - K * D) // D), (mm + K * D) // D + 1)
        j = j[(j >= 0) & (j < n_out)]
        i = j * D + K * D - mm
        cyc = FH * DT * D * j
        ref[j] += g[i] * np.exp(-2j * np.pi * (cyc - np.rint(cyc)))
        met[i] += 1
    assert np.all(met == 1)
    # taps at whole multiples of D are zero up to the sine's rounding
    assert np.all(np.abs(got - ref) <= 9 * 2.0 ** -24 * np.abs(ref) + 1e-15 * np.max(np.abs(g)))


@pytest.mark.parametrize("D,K", SHAPES)
def test_error_against_64_bits(gpu_lib, D, K):
    """White noise.  The taps' roundings (2^-24 / sqrt 3 rms each), the phase's (4 x 2^-24
    at most) and the sums': chains of at most Kd / 64 products and 8 additions, Kd = L + 7 D,
    each rounded by 2^-25 of a partial sum that is no larger than the output's
    rms, adding at random.  rms error <= (3 + sqrt(Kd / 64 + 8) / 2) 2^-24 of the rms
    output, and no output off by more than 6 times that.  Leaving out the tap half a
    zero spacing from the filter's end would be 14 times the bar on the rms or more."""
    import torch
    n_out = 3000
    torch.manual_seed(1000 * D + K)
    x = torch.randn(n_out * D, device="cuda")
    got = _run(gpu_lib, x, D, K, n_out).to(torch.complex128)
    g = torch.from_numpy(_taps(D, K)).cuda()
    L, c = len(g), K * D
    j = torch.arange(n_out, device="cuda")
    s = torch.zeros(n_out, dtype=torch.complex128, device="cuda")
    xp = torch.cat([torch.zeros(c, device="cuda"), x, torch.zeros(c + D, device="cuda")]).double()
    for i0 in range(0, L, 256):
        i = torch.arange(i0, min(i0 + 256, L), device="cuda")
        w = xp[j[:, None] * D + 2 * c - i[None, :]]
        s += (w * g[i].real).sum(1) + 1j * (w * g[i].imag).sum(1)
    cyc = FH * DT * D * j.double()
    ref = s * torch.exp(-2j * np.pi * (cyc - torch.round(cyc)))
    rms = ref.abs().square().mean().sqrt()
    err = (got - ref).abs() / rms
    bar = (3 + np.sqrt((L + 7 * D) / 64 + 8) / 2) * 2.0 ** -24
    print(f"D={D} K={K}: rms error {float(err.square().mean().sqrt()):.2e}, bar {bar:.2e}", flush=True)
    assert float(err.square().mean().sqrt()) <= bar and float(err.max()) <= 6 * bar


@pytest.mark.parametrize("D,K", SHAPES)
def test_bits_do_not_depend_on_the_length(gpu_lib, D, K):
    """The first outputs of a long series (few waves along the taps where the
    filter is short) and of its beginning alone (16 waves) are the same bits."""
    import torch
    torch.manual_seed(D + K)
    n_out, long_out = 2000, 300000
    x = torch.randn(long_out * D, device="cuda")
    whole = _run(gpu_lib, x, D, K, long_out)[:n_out]
    start = _run(gpu_lib, x[:n_out * D + K * D].contiguous(), D, K, n_out)
    assert torch.equal(torch.view_as_real(whole), torch.view_as_real(start))
