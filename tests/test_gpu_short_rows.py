"""The streaming boxcars on rows of a few steps (work-groups of 1, 2 and 3 waves,
rows walked from their first start or from a boundary of the outputs), with the
two outputs on different alignments, one of them, or neither: against the
register-window form of the same list (SPD_BOXCAR_FORM=window), the same SNRs
bit for bit and the same candidates; the width indices equal where the SNR is
not negative (between exactly equal negative SNRs the two keep different
maximisers)."""
import os

import numpy as np
import pytest
import torch

from paper_1611_09704_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


def run(x, n, col0, wcol0, pad, snr, widx):
    p = B.Params(list(range(1, n + 1)), 3.5)
    R, nout = x.shape[0], x.shape[1] - n + 1
    st = B.msd_compute(x, p)
    width = max(col0, wcol0) + nout + pad
    s = torch.full((R, width), -99.0, device=DEV)
    w = torch.full((R, width), 255, dtype=torch.uint8, device=DEV)
    cand, count = B.new_candidates(1 << 16, DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
    B.boxcar_snr(x, p, st, snr=s[:, col0:col0 + nout] if snr else None,
                 widx=w[:, wcol0:wcol0 + nout] if widx else None, cand=cand, cand_count=count)
    c = B.candidates_to_numpy(cand, int(count.item()))
    return s, w, c[np.lexsort((c["t"], c["row"]))]


@pytest.mark.parametrize("nout", [1, 3, 512, 513, 1024, 1500, 2047, 2048, 2600, 4100])
@pytest.mark.parametrize("col0,wcol0,snr,widx", [(0, 0, True, True), (3, 3, True, True), (3, 4, True, True),
                                                 (7, 1, True, False), (1, 7, False, True), (0, 0, False, False)])
def test_short_rows(nout, col0, wcol0, snr, widx):
    n, off, R = (8, 1, 37) if nout % 2 else (3, 0, 64)
    print("case: short rows nout=%d n=%d col0=%d wcol0=%d" % (nout, n, col0, wcol0), flush=True)
    g = torch.Generator(device=DEV).manual_seed(nout)
    x = torch.randn((R, off + nout + n - 1), generator=g, device=DEV)[:, off:]
    got = run(x, n, col0, wcol0, 2, snr, widx)
    os.environ["SPD_BOXCAR_FORM"] = "window"
    try:
        want = run(x, n, col0, wcol0, 2, True, True)
    finally:
        del os.environ["SPD_BOXCAR_FORM"]
    assert torch.equal(got[0], want[0] if snr else torch.full_like(got[0], -99.0))
    if widx:
        pos = torch.ones_like(want[1], dtype=torch.bool)                # canaries too
        pos[:, wcol0:wcol0 + nout] = want[0][:, col0:col0 + nout] >= 0
        assert torch.equal(got[1][pos], want[1][pos])
    else:
        assert torch.all(got[1] == 255)
    assert len(got[2]) > 0 or nout < 512
    for f in ("row", "t", "width", "snr"):
        assert np.array_equal(got[2][f], want[2][f])


def test_long_runs():
    """Candidates only, on enough rows for runs of 16 steps."""
    x = torch.randn((6144, 49153), generator=torch.Generator(device=DEV).manual_seed(1), device=DEV).to(torch.float16)
    p = B.Params(list(range(1, 9)), 6.0)
    st = B.msd_compute(x, p)
    print("case: long runs", flush=True)
    got = []
    for form in ("", "window"):
        os.environ["SPD_BOXCAR_FORM"] = form
        try:
            cand, count = B.new_candidates(1 << 16, DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
            B.boxcar_snr(x, p, st, cand=cand, cand_count=count)
            c = B.candidates_to_numpy(cand, int(count.item()))
            got.append(c[np.lexsort((c["t"], c["row"]))])
        finally:
            del os.environ["SPD_BOXCAR_FORM"]
    assert len(got[0]) > 0
    for f in ("row", "t", "width", "snr"):
        assert np.array_equal(got[0][f], got[1][f])
