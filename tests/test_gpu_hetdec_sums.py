"""The sums of the time-domain front end: an output's bits depend on the filter
and not on the length of the series."""
import pytest

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
