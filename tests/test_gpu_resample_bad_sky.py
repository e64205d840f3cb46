"""A sky row that is not a number: its series, positions and antenna sums are NaN
at every sampling interval, and the rows beside it are untouched."""
import numpy as np
import pytest

from paper_0912_4255_amd import synth
from tests.helpers import make_inputs, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gaps", [[], [[0, 40], [900, 1000]], [[100, 5000]]])
@pytest.mark.parametrize("binary", [False, True])
@pytest.mark.parametrize("dt", [0.5, 2.0, 4.0])
def test_nan_sky(gpu_lib, dt, binary, gaps):
    import torch
    w = synth.small_workload(n=5000, dt=dt, taps=16, nfft_policy=synth.NFFT_SMOOTH7)
    w.gaps = [np.array(gaps, dtype=np.int64).reshape(-1, 2)]
    xs, gs = make_inputs(w, seed=2)
    plan = gpu_lib.Plan(w)
    rows = np.array([[1.2, 0.3], [np.nan, 0.3], [1.2, np.nan], [1.2, 0.3]])
    if binary:
        plan.set_binary(True)
        rows = np.column_stack([rows, [[1.44, 68023.7, 2.3e4]] * 4])
    tx, tg = to_gpu(xs, gs)
    o = {k: v.cpu().numpy() for k, v in plan.resample(tx, tg, torch.from_numpy(rows).cuda())[0].items()}
    plan.close()
    for s in (1, 2):
        assert np.all(np.isnan(o["z"][s].real)) and np.all(np.isnan(o["tm"][s])) and np.all(np.isnan(o["u"][s]))
        # masked by sample 0: inside a gap nothing is summed
        seen = not (gaps and gaps[0][0] == 0)
        assert np.all(np.isnan(o["abc"][s])) if seen else np.all(o["abc"][s] == 0)
        bits = np.unpackbits(o["mask"][s].view(np.uint8), bitorder="little")[:w.segment.n]
        assert np.all(bits == seen)
    for k, v in o.items():
        assert np.array_equal(v[0], v[3]) and np.all(np.isfinite(v[0].real if np.iscomplexobj(v) else v[0]))
