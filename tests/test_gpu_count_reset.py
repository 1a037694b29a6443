"""The candidate count that a detection's merge resets, where a unit has more than
64 blocks (the merge by a work-group): a pass on a count that holds something
else finds what the pass before it found."""
import pytest
import torch

from paper_1611_09704_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("scope,R,L", [("row", 2, 65 * 16384), ("plane", 9, 8 * 16384)])
@pytest.mark.parametrize("static", [False, True])
def test_counts_are_reset_by_the_work_group_merge(scope, R, L, static):
    print("case: count reset %s %dx%d" % (scope, R, L), flush=True)
    x = torch.randn((R, L), generator=torch.Generator(device=DEV).manual_seed(R), device=DEV)
    p = B.Params(list(range(1, 9)), 4.0, scope)
    call = B.spd_detect_static if static else B.spd_detect
    cand, count = B.new_candidates(1 << 18, DEV), torch.full((1,), 77, dtype=torch.int64, device=DEV)
    n = []
    for k in range(3):
        call(x, p, cand=cand, cand_count=count)
        n.append(int(count.item()))
        count.fill_(1000 * k)
    assert n[0] == n[1] == n[2] > 0
    assert len(B.detect(x, list(range(1, 9)), 4.0, scope=scope)["cands"]) == n[0]
