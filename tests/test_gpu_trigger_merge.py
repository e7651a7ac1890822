"""The merge of a beam's triggers at the switch between one wave's registers (64
triggers at most) and the general path, exactly against the oracle: beams of 0,
1, 63, 64, 65 and 130 triggers, within one trial and over several, alone and side
by side, single and in chains."""
import numpy as np
import pytest

import oracle
from test_gpu_trigger import check_equal, make_cand, run_gpu_trigger
from paper_1612_06592_amd import lp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts", [(0,), (1,), (63,), (64,), (65,), (130,),
                                    (64, 65, 0, 63)])
@pytest.mark.parametrize("n_tec", [1, 5])
@pytest.mark.parametrize("gap", [2, 20])
def test_counts_around_one_wave(counts, n_tec, gap):
    rng = np.random.default_rng(sum(counts) * 100 + 10 * n_tec + gap)
    n_beams, n_t, frame0, k_sigma = len(counts), 4096, 5000, 2.0 + 1.0 / 512
    ns = n_beams * n_tec
    raw, sigma, wmax, warg = make_cand(rng, n_beams, n_tec, n_t, frame0,
                                       rng.integers(-2, 4, ns), 0.0, k_sigma)
    head = raw[:ns * n_t * 8].view(np.float32).reshape(ns, n_t, 2)
    for b, count in enumerate(counts):
        # One run of one or two windows each, `gap` windows after the last at
        # least, in a trial of its own choice: some runs chain, across trials
        # too, and each is one trigger of its series.
        at = 10
        for _ in range(count):
            q = b * n_tec + rng.integers(n_tec)
            for m in range(at, at + rng.integers(1, 3)):
                wmax[q, m] = sigma[q] * rng.integers(514, 1100) / 256.0
                head[q, m, 0] = wmax[q, m]
            at += gap + rng.integers(1, 10)
        fired = wmax[b * n_tec:(b + 1) * n_tec] > k_sigma * sigma[
            b * n_tec:(b + 1) * n_tec, None]
        assert (fired[:, 1:] & ~fired[:, :-1]).sum() == count
    trig, snr, best = oracle.trigger(sigma, wmax, warg, n_beams, n_tec, n_t,
                                     frame0, lp.WARM_FRAMES, k_sigma)
    g = run_gpu_trigger(raw, n_beams, n_tec, n_t, frame0, k_sigma, 400)
    check_equal(g, trig, 400)
    assert np.array_equal(g["snr"], snr.astype(np.float32))
    assert np.array_equal(g["best"], best)
