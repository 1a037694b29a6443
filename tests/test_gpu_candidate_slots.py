"""Candidates taken with one atomic per wave: from none to every start, from every
kernel that writes the list, with room for all of them and for fewer; and the
batch form's table of beams at its largest, 256 beams."""
import numpy as np
import pytest
import torch

from paper_1611_09704_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"
LISTS = {"stream": list(range(1, 9)), "stream 16": list(range(1, 17)), "window": list(range(1, 25)),
         "strided": [1, 2, 5, 9], "dit": list(range(1, 17)) + list(range(18, 33, 2))}


def triples(c):
    o = np.lexsort((c["t"], c["row"]))
    return c["row"][o], c["t"][o], c["width"][o], c["snr"][o]


@pytest.mark.parametrize("name", list(LISTS))
@pytest.mark.parametrize("thr", [-1e30, 0.5, 3.5, 1e30])
def test_list_against_stored_outputs(name, thr):
    print("case: slots %s thr=%g" % (name, thr), flush=True)
    W = LISTS[name]
    R, L = 5, 5003
    g = torch.Generator(device=DEV).manual_seed(len(W))
    x = torch.randn((R, L), generator=g, device=DEV)
    p = B.Params(W, thr)
    no = L - W[-1] + 1
    st = B.msd_compute(x, p)
    snr, widx = torch.empty((R, no), device=DEV), torch.empty((R, no), dtype=torch.uint8, device=DEV)
    for cap in (R * no, 100):
        cand = torch.full((cap + 1, B.CANDIDATE_DTYPE.itemsize), 0xAB, dtype=torch.uint8, device=DEV)
        count = torch.zeros(1, dtype=torch.int64, device=DEV)
        kw = dict(snr=snr, widx=widx, cand=cand[:cap], cand_count=count)
        if name == "dit":
            B.boxcar_snr_dit(x, p, 1, st, **kw)
        else:
            B.boxcar_snr(x, p, st, **kw)
        s, w = snr.cpu().numpy(), widx.cpu().numpy()
        row, t = np.nonzero(s >= np.float32(thr))
        want = (row, t, np.array(W)[w[row, t]], s[row, t])
        sel, seln = torch.full_like(cand, 0xAB), torch.zeros_like(count)
        B.select_candidates(snr, widx, p, cand=sel[:cap], cand_count=seln)
        for c, n in ((cand, count), (sel, seln)):
            assert int(n.item()) == len(row)
            assert torch.all(c[cap] == 0xAB)
            if cap >= len(row):
                for a, b in zip(triples(B.candidates_to_numpy(c, int(n.item()))), want):
                    assert np.array_equal(a, b)
            else:                                             # as many distinct ones as there is room for
                r, tt, ww, v = triples(B.candidates_to_numpy(c[:cap], cap))
                assert len(set(zip(r.tolist(), tt.tolist()))) == cap
                assert np.array_equal(v, s[r, tt]) and np.array_equal(ww, np.array(W)[w[r, tt]])


@pytest.mark.parametrize("W", [list(range(1, 25)), [1, 2, 5, 9]])
def test_most_beams(W):
    print("case: slots 256 beams n=%d" % len(W), flush=True)
    g = torch.Generator(device=DEV).manual_seed(5)
    p = B.Params(W, 3.0)
    beams = []
    for b in range(256):
        R, L = 1 + b % 3, 24 + (b * 37) % 4500
        x = torch.randint(0, 256, (R, L), generator=g, device=DEV, dtype=torch.uint8)
        beams.append((x, torch.full((R,), 0.5, device=DEV), torch.full((R,), 128.0, device=DEV)))
    plan = B.BatchPlan(beams, p, autotune=False)
    cand, count = B.new_candidates(1 << 18, DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
    plan.run(cand, count)
    got = B.candidates_to_numpy(cand, int(count.item()))
    n = 0
    for b, (x, sc, z) in enumerate(beams):
        c1, n1 = B.new_candidates(1 << 15, DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
        B.boxcar_snr(x, p, plan.stats(b), scale=sc, zero=z, cand=c1, cand_count=n1)
        for a, w in zip(triples(got[got["beam"] == b]), triples(B.candidates_to_numpy(c1, int(n1.item())))):
            assert np.array_equal(a, w)
        n += int(n1.item())
    assert n == len(got) > 0
