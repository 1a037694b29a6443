"""The streaming form of the short lists 1..n on rows at any offset: outputs of a
row that start off a 16-byte boundary (contiguous arrays of odd width, views
into wider ones), inputs at any element offset, one output only, candidates
only, and planes large enough for each run length.  Against the register-window
form of the same list (SPD_BOXCAR_FORM=window): the same SNRs bit for bit; the
width indices equal where the SNR is not negative (between exactly equal
negative SNRs the two keep different maximisers)."""
import os

import numpy as np
import pytest
import torch

from paper_1611_09704_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


def plane(R, L, dtype, off, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    if dtype == torch.uint8:
        x = torch.randint(0, 256, (R, L + off), generator=g, device=DEV, dtype=torch.uint8)
        return x[:, off:], torch.full((R,), 0.25, device=DEV), torch.full((R,), 120.0, device=DEV)
    x = torch.randn((R, L + off), generator=g, device=DEV).to(dtype)
    return x[:, off:], None, None


def run(x, sc, z, n, col0, pad, snr=True, widx=True, cap=1 << 18, thr=4.5):
    p = B.Params(list(range(1, n + 1)), thr)
    R, nout = x.shape[0], x.shape[1] - n + 1
    st = B.msd_compute(x, p, scale=sc, zero=z)
    s = torch.full((R, col0 + nout + pad), -99.0, device=DEV)
    w = torch.full((R, col0 + nout + pad), 255, dtype=torch.uint8, device=DEV)
    cand, count = B.new_candidates(cap, DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
    B.boxcar_snr(x, p, st, scale=sc, zero=z, snr=s[:, col0:col0 + nout] if snr else None,
                 widx=w[:, col0:col0 + nout] if widx else None, cand=cand, cand_count=count)
    c = B.candidates_to_numpy(cand, int(count.item()))
    return s, w, c[np.lexsort((c["t"], c["row"]))]


def check(R, L, dtype, n, off=0, col0=0, pad=0, snr=True, widx=True, thr=4.5):
    print("case: stream R=%d L=%d %s n=%d off=%d col0=%d pad=%d" % (R, L, dtype, n, off, col0, pad), flush=True)
    x, sc, z = plane(R, L, dtype, off, seed=n + L)
    got = run(x, sc, z, n, col0, pad, snr, widx, thr=thr)
    os.environ["SPD_BOXCAR_FORM"] = "window"
    try:
        want = run(x, sc, z, n, col0, pad, thr=thr)
    finally:
        del os.environ["SPD_BOXCAR_FORM"]
    assert torch.equal(got[0], want[0] if snr else torch.full_like(got[0], -99.0))
    if widx:
        pos = want[0] >= 0
        pos[:, :col0], pos[:, want[0].shape[1] - pad:] = True, True        # canaries too
        assert torch.equal(got[1][pos], want[1][pos])
    else:
        assert torch.all(got[1] == 255)
    for f in ("row", "t", "width", "snr"):
        assert np.array_equal(got[2][f], want[2][f])


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.uint8])
@pytest.mark.parametrize("n", [1, 2, 5, 8, 12, 15, 16])
def test_lists(dtype, n):
    check(19, 2048 + 13, dtype, n, off=n % 4)


@pytest.mark.parametrize("dtype", [torch.float32, torch.uint8])
@pytest.mark.parametrize("L", [16, 17, 511, 527, 528, 1024 + 15, 1024 + 16, 4096 + 31, 9001])
def test_lengths_and_offsets(dtype, L):
    check(33, L, dtype, 16, off=1)
    check(17, L, dtype, 16, off=2, col0=L % 16, pad=5)


@pytest.mark.parametrize("snr,widx", [(True, False), (False, True), (False, False)])
def test_single_outputs(snr, widx):
    check(9, 6001, torch.float32, 16, off=3, col0=3, pad=2, snr=snr, widx=widx)


def test_run_lengths():
    check(16, 4100, torch.float32, 8)                   # 2 steps a run
    check(1024, 33000, torch.float32, 16, off=1, thr=5.5)        # 4
    check(4096, 32801, torch.uint8, 16, off=1, thr=9.0)          # 8
