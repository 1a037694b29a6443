"""The merge of block partials over a few lanes per unit, at the edges of its
lane counts (1, 2, 3, 4, 63, 64 blocks per unit, and 65 beyond it) and with
units that do not fill a wave.  8-bit samples have exact integer partials, so
mean, sigma and the widest boxcar's sigma agree with 64-bit NumPy to the few
roundings of the merges: at most 65 merges of about 10 operations, 65 * 10 *
1.1e-16 = 7e-14, and NumPy's own sums; 1e-11 is asked for.  The candidate count,
which the merge resets, comes out the same on a second pass without a reset in
between."""
import numpy as np
import pytest
import torch

from paper_1611_09704_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"
BLOCK, BATCH_BLOCK = 16384, 32768
RTOL = 1e-11


def plane(R, L, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randint(0, 256, (R, L), generator=g, device=DEV, dtype=torch.uint8)
    return x, torch.full((R,), 0.25, device=DEV), torch.full((R,), 120.0, device=DEV)


def want(x, w):
    v = (x.cpu().numpy().astype(np.float64) - 120.0) * 0.25
    c = np.cumsum(np.pad(v, ((0, 0), (1, 0))), axis=1)          # exact: quarters below 2^53
    return v, c[:, w:] - c[:, :-w]


def check(st, v, y):
    st = st.cpu().numpy()
    np.testing.assert_allclose(st[:, 1], v.std(axis=1), rtol=RTOL)
    np.testing.assert_allclose(st[:, 2], y.std(axis=1), rtol=RTOL)
    assert np.all(np.abs(st[:, 0] - v.mean(axis=1)) <= RTOL * v.std(axis=1))


@pytest.mark.parametrize("blocks,R", [(1, 1), (1, 130), (2, 33), (3, 17), (4, 64), (63, 3), (64, 2), (65, 2)])
def test_units(blocks, R):
    print("case: finalize blocks=%d R=%d" % (blocks, R), flush=True)
    x, sc, z = plane(R, blocks * BLOCK - 5, seed=blocks)
    p = B.Params([1, 2, 3, 7], 4.0, "row", "linear")
    v, y = want(x, 7)
    state = torch.zeros((R, 6), dtype=torch.float64, device=DEV)
    st = B.msd_compute(x, p, scale=sc, zero=z, state=state)
    check(st, v, y)
    assert np.array_equal(state.cpu().numpy()[:, 0], np.full(R, x.shape[1]))
    one = B.msd_compute(x, B.Params([1, 2, 3, 7], 4.0, "plane", "linear"), scale=sc, zero=z)   # one unit of R * blocks
    check(one, v.reshape(1, -1), y.reshape(1, -1))


def test_counts_are_reset():
    x, sc, z = plane(9, 3 * BLOCK, seed=2)
    W = list(range(1, 25))
    p = B.Params(W, 3.0)
    cand, count = B.new_candidates(1 << 18, DEV), torch.full((1,), 77, dtype=torch.int64, device=DEV)
    stats = torch.empty((9, B.STATS_FIELDS), dtype=torch.float64, device=DEV)
    need = B.msd_compute(x, p, scale=sc, zero=z)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=DEV)
    n = []
    for _ in range(2):
        B.spd_detect(x, p, scale=sc, zero=z, stats=stats, cand=cand, cand_count=count, workspace=ws)
        n.append(int(count.item()))
    assert n[0] == n[1] > 0 and torch.equal(stats, need)


@pytest.mark.parametrize("shapes", [[(3, 900), (1, 40), (70, 1000)], [(5, BATCH_BLOCK + 1), (2, 100), (9, 5 * BATCH_BLOCK)],
                                    [(2, 64 * BATCH_BLOCK), (3, 500)], [(1, 65 * BATCH_BLOCK), (2, 500)]])
@pytest.mark.parametrize("graph", [False, True])
def test_batch(shapes, graph):
    print("case: finalize batch %s graph=%s" % (shapes, graph), flush=True)
    beams = [plane(R, L, seed=k) for k, (R, L) in enumerate(shapes)]
    p = B.Params(list(range(1, 25)), 3.5, "row", "linear")
    plan = B.BatchPlan(beams, p, autotune=False)
    cand, count = B.new_candidates(1 << 18, DEV), torch.full((1,), 5, dtype=torch.int64, device=DEV)
    n = []
    for _ in range(3):
        plan.run(cand, count, use_graph=graph)
        torch.cuda.synchronize()
        n.append(int(count.item()))
    assert n[0] == n[1] == n[2] > 0
    for b, (x, _, _) in enumerate(beams):
        check(plan.stats(b), *want(x, 24))
