"""First-pass rows on workgroups of 128, 256 and 512 threads, general stages and
run-time row plans: 2F against the oracle at sampled bins (the bar of the
full-band tests), and the same bits in plain mode, in batched mode and whatever
number of spindowns shares a row."""
import numpy as np
import pytest

from oracle import fstat as of
from paper_0912_4255_amd import synth
from paper_0912_4255_amd.api import plan_desc_from_workload
from tests.helpers import make_inputs, to_gpu, twoF_tol

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l1,l2", [
    (24, 512),       # shorter than a workgroup: general stages, 128 threads
    (400, 512),
    (1350, 256),     # at most 256 columns: 256 threads
    (1568, 100),
    (3125, 64),      # 5^5, odd: the rows do not end below L1 / 2
    (6000, 32),      # 512 threads
    (900, 768),      # run-time row plans from here: 128 threads
    (1960, 512),     # 256
    (4320, 256),
])
def test_rows_against_oracle_and_batching(gpu_lib, l1, l2):
    import torch
    n = l1 * l2 // 2
    w = synth.small_workload(n=n, dt=1.0, kernel=synth.KERNEL_LANCZOS, taps=8)
    xs, gaps = make_inputs(w, seed=l1)
    d = plan_desc_from_workload(w)
    d.fft_l1 = l1
    plan = gpu_lib.Plan(desc=d)
    assert (plan.fft_l1, plan.fft_l2) == (l1, l2)
    tx, tg = to_gpu(xs, gaps)
    sky = torch.tensor([[1.0, 0.2]], dtype=torch.float64).cuda()
    fdots = np.array([-3e-10, 0.0, -1e-9])
    fd = torch.from_numpy(fdots).cuda()
    got = plan.fstat(tx, tg, sky, fd)
    assert torch.equal(got, plan.fstat(tx, tg, sky, fd, mode=gpu_lib.RSF_MODE_PLAIN))
    plan.set_batching(2, 3)
    assert torch.equal(got, plan.fstat(tx, tg, sky, fd))
    plan.close()
    got = got.cpu().numpy()
    rss = [of.resample(xs[0], gaps[0], w.segment, 1.0, 0.2, w.eph, w.detectors[0], w.kernel, w.taps)]
    rng = np.random.default_rng(l2)
    idx = np.unique(np.concatenate([[0, 1, plan.n_out // 2, plan.n_out - 1], rng.integers(0, plan.n_out, 28)]))
    for i, f in enumerate(fdots):
        ref = of.fstat_bins(rss, w.detectors, f, plan.n_fft, plan.s_lo + idx)
        assert np.all(np.abs(got[i][idx] - ref) <= twoF_tol(ref)), (l1, l2, i)
