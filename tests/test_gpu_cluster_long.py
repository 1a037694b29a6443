"""Peak finding over lists around the length from which launches with wide windows
use twice the work-groups (262,144 entries, windows of 1,024 samples or more):
the peaks among the list's first n entries, against a max filter.  SNRs are
distinct, so no tie rule enters."""
import numpy as np
import pytest
import torch

from paper_1611_09704_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("radii", [(0, 511), (0, 512), (4, 60), (16, 15)])      # 1,023, 1,025, 1,089, 1,023 samples
@pytest.mark.parametrize("n", [1, 262143, 262144, 262145, 320000])
def test_long_lists(n, radii):
    R, L = 40, 8000
    print("case: long list n=%d radii=%s" % (n, radii), flush=True)
    g = torch.Generator(device=DEV).manual_seed(3)
    snr = torch.randperm(R * L, generator=g, device=DEV).to(torch.float32).reshape(R, L)
    widx = torch.zeros((R, L), dtype=torch.uint8, device=DEV)
    cand, count = B.new_candidates(R * L, DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
    B.select_candidates(snr, widx, B.Params([1], -1.0), cand=cand, cand_count=count)
    assert int(count.item()) == R * L
    count.fill_(n)
    best = torch.nn.functional.max_pool2d(snr[None, None], (2 * radii[0] + 1, 2 * radii[1] + 1), 1, radii)[0, 0]
    peak = (snr == best).cpu().numpy()
    first = B.candidates_to_numpy(cand, n)
    want = sorted((int(r), int(t)) for r, t in zip(first["row"], first["t"]) if peak[r, t])
    peaks, got_n = B.cluster_candidates(snr, cand, count, *radii)
    got = B.candidates_to_numpy(peaks, int(got_n.item()))
    assert sorted(zip(got["row"].tolist(), got["t"].tolist())) == want
    assert len(want) > 0 or n == 1
