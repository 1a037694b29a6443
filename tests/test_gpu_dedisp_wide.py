"""The wide layout of the de-dispersion (16-byte entries of 8 starts, 16-bit
partial sums) against the matrix form, the chunk-by-chunk kernel and the oracle.
Lists of 3 to 4 samples a trial take it by themselves, any list it fits with
SPD_DEDISP_FORM=wide.  Channel counts sit around the 16 of a chunk and the 256 of
a flush of the partial sums; saturated input over 4,096 channels overflows 16
bits after 257 channels unless every flush is made."""
import os

import numpy as np
import pytest
import torch

import oracle
from paper_1611_09704_amd import binding as B
from paper_1611_09704_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def run(plan, fb, form):
    os.environ["SPD_DEDISP_FORM"] = form
    try:
        buf = torch.full((plan.n_dm, fb.shape[1] - plan.max_delay + 3), -7.0, device=DEV)
        y = plan.run(fb, out=buf)
        torch.cuda.synchronize()
    finally:
        del os.environ["SPD_DEDISP_FORM"]
    assert torch.all(buf[:, y.shape[1]:] == -7.0), "wrote past n_out"
    return y


@pytest.mark.parametrize("C", [1, 15, 16, 17, 240, 255, 256, 257, 272, 511, 512, 513, 1030])
@pytest.mark.parametrize("step", [1.0, 3.5])
def test_forms_agree(C, step):
    n_dm, S = 19, 1700
    band = (1500.0, 100.0 / C, 64e-6)
    kc = oracle.dedisp_channel_factors(C, *band)
    dm = np.arange(n_dm) * step / max(kc[-1], 1e-9)
    print("case: dedisp wide C=%d step=%g" % (C, step), flush=True)
    fb = synth.filterbank(C, S, seed=900 + C, device=DEV)
    plan = B.DedispPlan(C, *band, dm)
    want = oracle.dedisperse(fb.cpu().numpy(), dm, kc)
    for form in ("wide", "generic", ""):
        assert np.array_equal(run(plan, fb, form).cpu().numpy().astype(np.float64), want), form


@pytest.mark.parametrize("step", [1.0, 3.5])
def test_saturated_sums(step):
    C, S = 4096, 1400
    band = (1550.0, 300.0 / C, 64e-6)
    kc = oracle.dedisp_channel_factors(C, *band)
    plan = B.DedispPlan(C, *band, np.arange(20) * step / kc[-1])
    fb = torch.full((C, S), 255, dtype=torch.uint8, device=DEV)
    print("case: dedisp wide saturated step=%g" % step, flush=True)
    for form in ("wide", "generic", ""):
        assert torch.all(run(plan, fb, form) == 255.0 * C), form
