"""Peak finding with many peaks per wave (noise, where most candidates are peaks):
the peak set and count against a max filter, and a peak list with room for
fewer.  SNRs are distinct, so no tie rule enters."""
import numpy as np
import pytest
import torch

from paper_1611_09704_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("radii", [(0, 0), (1, 2), (2, 9)])
@pytest.mark.parametrize("R,L,thr", [(1, 70, -9.0), (7, 4099, 1.0), (64, 33000, 2.0), (200, 30000, -9.0)])
def test_many_peaks(R, L, thr, radii):
    print("case: many peaks %dx%d thr=%g radii=%s" % (R, L, thr, radii), flush=True)
    g = torch.Generator(device=DEV).manual_seed(R)
    snr = torch.randperm(R * L, generator=g, device=DEV).to(torch.float32).reshape(R, L) / (R * L) * 8 - 4
    widx = torch.zeros((R, L), dtype=torch.uint8, device=DEV)
    cand, count = B.new_candidates(R * L, DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
    B.select_candidates(snr, widx, B.Params([1], thr), cand=cand, cand_count=count)
    best = torch.nn.functional.max_pool2d(snr[None, None], (2 * radii[0] + 1, 2 * radii[1] + 1), 1, radii)[0, 0]
    want = torch.nonzero((snr == best) & (snr >= thr)).cpu().numpy()
    for cap in (R * L, 10):
        peaks, n = torch.full((cap + 1, B.CANDIDATE_DTYPE.itemsize), 0xAB, dtype=torch.uint8, device=DEV), torch.zeros_like(count)
        B.cluster_candidates(snr, cand, count, *radii, peaks=peaks[:cap], peak_count=n)
        assert int(n.item()) == len(want)
        assert torch.all(peaks[cap] == 0xAB)
        got = B.candidates_to_numpy(peaks[:cap], min(cap, len(want)))
        pairs = sorted(zip(got["row"].tolist(), got["t"].tolist()))
        all_ = [tuple(w) for w in want.tolist()]
        assert pairs == all_ if cap >= len(all_) else set(pairs) <= set(all_) and len(set(pairs)) == cap
