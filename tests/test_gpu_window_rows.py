"""The register-window form of grouped width lists on rows at any offset: lists
that step by 1 throughout (1..8k) and mixed ones, every input type, windows
shorter and longer than the samples loaded ahead (1,024), rows around the edges
of a tile, lists whose last group of 8 is not full, zero variance and
non-finite samples.  Against the strided form of the same list (SPD_BOXCAR_FORM=strided),
which has its own staging and sums in the same order: everything bit for bit."""
import os

import numpy as np
import pytest
import torch

from paper_1611_09704_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"
MIXED = list(range(1, 33)) + list(range(34, 65, 2))          # groups of step 1, then of step 2
LISTS = {"1..24": list(range(1, 25)), "1..32": list(range(1, 33)), "1..128": list(range(1, 129)),
         "1..256": list(range(1, 257)), "mixed": MIXED}


def plane(R, L, dtype, off, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    if dtype == torch.uint8:
        x = torch.randint(0, 256, (R, L + off), generator=g, device=DEV, dtype=torch.uint8)
        return x[:, off:], torch.full((R,), 0.25, device=DEV), torch.full((R,), 120.0, device=DEV)
    x = torch.randn((R, L + off), generator=g, device=DEV).to(dtype)
    return x[:, off:], None, None


def run(x, sc, z, W):
    p = B.Params(W, 4.0)
    st = B.msd_compute(x, p, scale=sc, zero=z)
    R, nout = x.shape[0], x.shape[1] - W[-1] + 1
    snr = torch.full((R, nout + 1), -99.0, device=DEV)
    widx = torch.full((R, nout + 1), 255, dtype=torch.uint8, device=DEV)
    cand, count = B.new_candidates(1 << 17, DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
    B.boxcar_snr(x, p, st, scale=sc, zero=z, snr=snr[:, :nout], widx=widx[:, :nout], cand=cand, cand_count=count)
    c = B.candidates_to_numpy(cand, int(count.item()))
    return snr, widx, c[np.lexsort((c["t"], c["row"]))]


def check(R, L, dtype, W, off):
    print("case: window R=%d L=%d %s n=%d off=%d" % (R, L, dtype, len(W), off), flush=True)
    x, sc, z = plane(R, L, dtype, off, seed=len(W) + L)
    got = run(x, sc, z, W)
    os.environ["SPD_BOXCAR_FORM"] = "strided"
    try:
        want = run(x, sc, z, W)
    finally:
        del os.environ["SPD_BOXCAR_FORM"]
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    for f in ("row", "t", "width", "snr"):
        assert np.array_equal(got[2][f], want[2][f])


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.uint8])
@pytest.mark.parametrize("name", list(LISTS))
def test_lists_at_any_offset(dtype, name):
    W = LISTS[name]
    for off in range(4):
        check(5, 4111 + W[-1], dtype, W, off)


@pytest.mark.parametrize("dtype", [torch.float32, torch.uint8])
@pytest.mark.parametrize("extra", [0, 1, 7, 511, 512, 520, 2047, 2048, 2049])
def test_tile_edges(dtype, extra):
    for W in (LISTS["1..32"], MIXED):
        check(3, W[-1] + extra, dtype, W, 1)


SHORT = {"1..17": list(range(1, 18)), "1..23": list(range(1, 24)), "1..100": list(range(1, 101)),
         "1..255": list(range(1, 256)), "mixed 35": (list(range(1, 17)) + list(range(18, 80, 2)))[:35],
         "2,4,6": [2, 4, 6], "step 2, 13": list(range(2, 28, 2))}


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.uint8])
@pytest.mark.parametrize("name", list(SHORT))
def test_short_last_group(dtype, name):
    W = SHORT[name]
    for extra in (0, 1, 512, 2048, 4111):
        check(3, W[-1] + extra, dtype, W, 1)


def test_short_last_group_special_values():
    print("case: window special values", flush=True)
    W = list(range(1, 21))
    for scope in ("row", "plane"):
        x = torch.randn((6, 3000), device=DEV)
        x[1] = 0.25                                           # zero variance
        x[2, 700] = float("inf")
        x[3, 900] = float("-inf")
        x[4, 1000:1003] = float("nan")
        x[5] = -0.0
        p = B.Params(W, 4.0, scope)
        st = torch.tensor([[0.0, 1.0, 0.0, 0.0, 0.0]] * 6, dtype=torch.float64, device=DEV)
        st[1] = B.msd_compute(x[1:2].contiguous(), p)[0]
        out = []
        for form in ("", "strided"):
            os.environ["SPD_BOXCAR_FORM"] = form
            try:
                s, w = torch.zeros((6, 2981), device=DEV), torch.zeros((6, 2981), dtype=torch.uint8, device=DEV)
                B.boxcar_snr(x, p, st, snr=s, widx=w)
                out.append((s, w))
            finally:
                del os.environ["SPD_BOXCAR_FORM"]
        (s, w), (s2, w2) = out
        assert torch.equal(torch.isnan(s), torch.isnan(s2)) and torch.equal(torch.nan_to_num(s), torch.nan_to_num(s2))
        assert torch.equal(w, w2)
