"""De-dispersions of few channels or few trials: the form and work-groups that the
library chooses are not slower than the wide layout, which it could take instead
(SPD_DEDISP_FORM=wide).  Where the matrix form stored its sums 16 bytes at a time,
or ran 64-trial work-groups on a handful of trials, it took 1.3 to 2.4 times as
long; the bound of 1.25 leaves room for the spread of short kernels."""
import os

import numpy as np
import pytest
import torch

import oracle
from paper_1611_09704_amd import binding as B
from paper_1611_09704_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def best_ms(plan, fb, out):
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    best = float("inf")
    for _ in range(6):
        torch.cuda.synchronize()
        e[0].record()
        for _ in range(20):
            plan.run(fb, out=out)
        e[1].record()
        torch.cuda.synchronize()
        best = min(best, e[0].elapsed_time(e[1]) / 20)
    return best


@pytest.mark.parametrize("C,n_dm,n_out", [(4, 128, 1 << 18), (16, 64, 1 << 18), (4, 1, 1 << 20), (16, 16, 1 << 20),
                                          (32, 8, 1 << 20), (64, 24, 1 << 20), (48, 16, 1 << 18)])
def test_chosen_form_is_not_slower_than_the_wide_layout(C, n_dm, n_out):
    band = (1550.0, 300.0 / C, 64e-6)
    kc = oracle.dedisp_channel_factors(C, *band)
    plan = B.DedispPlan(C, *band, [i / kc[-1] for i in range(n_dm)])
    S = (n_out + plan.max_delay + 3) // 4 * 4
    fb = torch.randint(0, 256, (C, S), dtype=torch.uint8, device=DEV)
    out = torch.empty((n_dm, S - plan.max_delay), device=DEV)
    chosen = best_ms(plan, fb, out)
    os.environ["SPD_DEDISP_FORM"] = "wide"
    try:
        wide = best_ms(plan, fb, out)
    finally:
        del os.environ["SPD_DEDISP_FORM"]
    print("case: dedisp C=%d n_dm=%d n_out=%d chosen %.1f us wide %.1f us" % (C, n_dm, n_out, chosen * 1e3, wide * 1e3),
          flush=True)
    assert chosen <= 1.25 * wide


@pytest.mark.parametrize("C,n_dm,n_out,step", [(2, 16, 524288, 1.0), (17, 13, 524289, 1.0), (9, 16, 524800, 2.0),
                                               (8, 5, 600001, 0.4), (3, 32, 400000, 1.0)])
def test_sums_of_few_trials(C, n_dm, n_out, step):
    """The 16-trial work-groups on a list they take for its length, and the edges beside it."""
    band = (1550.0, 300.0 / C, 64e-6)
    kc = oracle.dedisp_channel_factors(C, *band)
    dm = np.arange(n_dm) * step / kc[-1]
    plan = B.DedispPlan(C, *band, dm)
    print("case: dedisp few trials C=%d n_dm=%d n_out=%d" % (C, n_dm, n_out), flush=True)
    fb = synth.filterbank(C, n_out + plan.max_delay, seed=C + n_dm, device=DEV)
    out = torch.full((n_dm, n_out + 5), -7.0, device=DEV)
    y = plan.run(fb, out=out)
    assert torch.all(out[:, n_out:] == -7.0)
    assert np.array_equal(y.cpu().numpy().astype(np.float64), oracle.dedisperse(fb.cpu().numpy(), dm, kc))
