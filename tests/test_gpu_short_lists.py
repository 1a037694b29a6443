"""Lists of up to 16 widths in groups that step by 1 or 2, the last one short.  On
one plane they take the strided form; the register-window form, which batched
runs use for them, is made to take them here (SPD_BOXCAR_FORM=window).  On finite
samples both give the same bits; where every SNR is NaN the strided form, and so
the default, returns NaN."""
import os

import numpy as np
import pytest
import torch

from paper_1611_09704_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"
LISTS = {"2,4": [2, 4], "2,4,6": [2, 4, 6], "step 2, 7": list(range(2, 16, 2)), "step 2, 9": list(range(2, 20, 2)),
         "step 2, 15": list(range(2, 32, 2)), "1..8,10,12": list(range(1, 9)) + [10, 12],
         "1..8, step 2 to 22": list(range(1, 9)) + list(range(10, 24, 2))}


def run(x, W, form, st=None):
    p = B.Params(W, 3.5)
    st = B.msd_compute(x, p) if st is None else st
    nout = x.shape[1] - W[-1] + 1
    s = torch.full((x.shape[0], nout + 1), -99.0, device=DEV)
    w = torch.full((x.shape[0], nout + 1), 255, dtype=torch.uint8, device=DEV)
    cand, count = B.new_candidates(1 << 17, DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
    os.environ["SPD_BOXCAR_FORM"] = form
    try:
        B.boxcar_snr(x, p, st, snr=s[:, :nout], widx=w[:, :nout], cand=cand, cand_count=count)
    finally:
        del os.environ["SPD_BOXCAR_FORM"]
    c = B.candidates_to_numpy(cand, int(count.item()))
    return s, w, c[np.lexsort((c["t"], c["row"]))]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("name", list(LISTS))
def test_forms_agree(dtype, name):
    W = LISTS[name]
    for extra in (0, 1, 512, 2048, 4111):
        print("case: short list %s extra=%d" % (name, extra), flush=True)
        g = torch.Generator(device=DEV).manual_seed(extra)
        x = torch.randn((3, W[-1] + extra + 1), generator=g, device=DEV).to(dtype)[:, 1:]
        want = run(x, W, "strided")
        for form in ("", "window"):
            got = run(x, W, form)
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
            for f in ("row", "t", "width", "snr"):
                assert np.array_equal(got[2][f], want[2][f])


@pytest.mark.parametrize("name", list(LISTS))
def test_no_snr_is_nan(name):
    W = LISTS[name]
    print("case: short list %s NaN" % name, flush=True)
    x = torch.randn((4, 2500), generator=torch.Generator(device=DEV).manual_seed(2), device=DEV)
    x[1] = float("nan")
    x[2, 700:1400] = float("nan")
    st = B.msd_compute(x, B.Params(W, 3.5))
    st[2] = st[0]
    (s, w, _), (s2, w2, _) = run(x, W, "", st), run(x, W, "strided", st)
    assert torch.all(torch.isnan(s[1, :2500 - W[-1] + 1])) and torch.all(torch.isnan(s[2, 700:1390 - W[-1]]))
    assert torch.equal(torch.isnan(s), torch.isnan(s2))
    assert torch.equal(torch.nan_to_num(s), torch.nan_to_num(s2)) and torch.equal(w, w2)
