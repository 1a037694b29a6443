"""The matrix form of the de-dispersion (spd_dedisperse on fine DM lists) against
the oracle: sums of 8-bit samples are whole numbers, so every output must be
equal exactly.  Sizes sit at the edges of its tiles: trials around the quads of
4 and the 32- and 64-trial work-groups, channels around the 8 of a product,
starts around the 512 and 1,024 of a work-group, rows whose last dword is
partial, trials up to the most delay that the close and the far form take (4 and
9 samples over 4 trials) and one step past each, and lists whose quads are tight
but far apart (the 16-trial work-groups)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1611_09704_amd import binding as B
from paper_1611_09704_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def check(C, n_out, steps, pad=3):
    """steps: delay of each trial at the lowest channel, in samples."""
    band = (1550.0, 300.0 / C, 64e-6)
    kc = oracle.dedisp_channel_factors(C, *band)
    dm = np.asarray(steps, dtype=np.float64) / kc[-1]
    S = n_out + int(oracle.dedisp_delays(dm, kc).max())
    print("case: dedisp matrix C=%d n_dm=%d n_out=%d S=%d" % (C, dm.size, n_out, S), flush=True)
    fb = synth.filterbank(C, S, seed=C + n_out, device=DEV)
    plan = B.DedispPlan(C, *band, dm)
    buf = torch.full((dm.size, n_out + pad), -7.0, device=DEV)
    y = plan.run(fb, out=buf)
    torch.cuda.synchronize()
    assert y.shape[1] == n_out and torch.all(buf[:, n_out:] == -7.0)
    assert np.array_equal(y.cpu().numpy().astype(np.float64), oracle.dedisperse(fb.cpu().numpy(), dm, kc))


@pytest.mark.parametrize("C", [2, 7, 8, 9, 17])
@pytest.mark.parametrize("n_dm", [1, 4, 5, 31, 33, 65])
def test_channels_and_trials(C, n_dm):
    check(C, 700, np.arange(n_dm))


@pytest.mark.parametrize("n_out", [1, 2, 511, 512, 513, 1023, 1025, 1538])
def test_starts(n_out):
    check(24, n_out, np.arange(37) * 0.77)


@pytest.mark.parametrize("step", [0.0, 0.1, 1.0, 1.33, 1.34, 2.0, 2.66, 2.99, 3.0, 3.7])
def test_trial_spacing(step):
    check(40, 1300, np.arange(70) * step)


@pytest.mark.parametrize("step", [1.0, 1.9])
def test_large_work_groups(step):
    # 200 and 130 trials over enough starts that the 64-trial work-groups run
    check(11, 60001, np.arange(200 if step == 1.0 else 130) * step)


def test_tight_quads_far_apart():
    check(33, 900, np.concatenate([q * 35 + np.arange(4) for q in range(9)]))
    check(33, 900, np.concatenate([q * 35 + np.arange(4) * 2.5 for q in range(9)]))
