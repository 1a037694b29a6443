"""A server that de-disperses a fine list of trials (one sample of delay a trial, so
the matrix form runs on its staged planes, from the first chunk's and from the
carried halo's columns, into rows that start behind the detection halo), against
the streaming oracle over the oracle's de-dispersion of the whole series."""
import numpy as np
import pytest
import torch

import oracle
from paper_1611_09704_amd import binding as B
from paper_1611_09704_amd import synth
import spd_check as C
from test_gpu_serve import _drain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_dm,step,wmax", [(40, 1.0, 32), (38, 1.0, 16), (34, 2.0, 24)])
def test_server_with_fine_trials_matches_streaming_oracle(n_dm, step, wmax):
    C_ch, Lc, K, nb = 32, 3000, 3, 2
    band = (1500.0, 40.0 / C_ch, 64e-6)
    kc = oracle.dedisp_channel_factors(C_ch, *band)
    dm = np.arange(n_dm) * (step / kc[-1])
    W, thr = list(range(1, wmax + 1)), 6.0
    H = wmax - 1
    plan = B.DedispPlan(C_ch, *band, dm)
    md = plan.max_delay
    assert md % 4 != 0                                        # the view after chunk 0 starts early
    delays = oracle.dedisp_delays(dm, kc)
    rng = np.random.default_rng(77)
    fulls, chunks = [], []
    for b in range(nb):
        fb = synth.filterbank(C_ch, K * Lc, seed=800 + b, device="cuda")
        for k in range(1, K):                                 # pulses whose de-dispersed start straddles a cut
            synth.inject_along(fb, delays[int(rng.integers(0, n_dm))], k * Lc - md - 5, 12, 25)
        fulls.append(fb.cpu().numpy())
        chunks.append([fb[:, k * Lc:(k + 1) * Lc].contiguous().cpu().pin_memory() for k in range(K)])
    print("case: serve fine dedisp n_dm=%d step=%g md=%d" % (n_dm, step, md), flush=True)
    srv = B.Server(nb, C_ch, Lc, B.Params(W, thr), cand_capacity=8192, dedisp=plan)
    for k in range(K):
        for b in range(nb):
            srv.submit(b, k, chunks[b][k])
    results = _drain(srv, nb * K)
    srv.close()
    by = {(r["beam"], r["seq"]): (r, c) for r, c in results}
    for b in range(nb):
        y = oracle.dedisperse(fulls[b], dm, kc)
        state, n_found = None, 0
        for k in range(K):
            s0 = 0 if k == 0 else k * Lc - md
            lead = 0 if k == 0 else H
            view, toff = y[:, s0 - lead:(k + 1) * Lc - md], s0 - lead
            state, st, snr, widx = oracle.stream_step(view, W, new_col_begin=lead, state=state, sigma_mode="sqrtn")
            oc = oracle.select(snr, widx, W, thr, t_offset=toff)
            r, c = by[(b, k)]
            assert r["status"] == 0 and r["t_offset"] == toff, (b, k, r["t_offset"], toff)
            C.check_candidates(c, oc, thr, lambda row, t: snr[row, t - toff], C.width_rule(view, W, st, t_offset=toff))
            n_found += len(c)
        assert n_found > 0
