"""More series than the chip has CUs, with hundreds of triggers each and with
few, one trial and several: the lists are the oracle's, exactly."""
import numpy as np
import pytest

import oracle
from test_gpu_trigger import check_equal, make_cand, run_gpu_trigger
from paper_1612_06592_amd import lp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_beams,n_tec", [(300, 1), (520, 1), (200, 3)])
@pytest.mark.parametrize("fire", [0.003, 0.3])
def test_many_series_equal_oracle(n_beams, n_tec, fire):
    rng = np.random.default_rng(n_beams + n_tec)
    n_t, frame0, k_sigma, ns = 2048, 5000, 2.0 + 1.0 / 512, n_beams * n_tec
    raw, sigma, wmax, warg = make_cand(rng, n_beams, n_tec, n_t, frame0,
                                       rng.integers(-2, 4, ns), fire, k_sigma)
    trig, snr, best = oracle.trigger(sigma, wmax, warg, n_beams, n_tec, n_t,
                                     frame0, lp.WARM_FRAMES, k_sigma)
    cap = len(trig) + 1
    g = run_gpu_trigger(raw, n_beams, n_tec, n_t, frame0, k_sigma, cap)
    check_equal(g, trig, cap)
    assert np.array_equal(g["snr"], snr.astype(np.float32))
    assert np.array_equal(g["best"], best)
    assert np.array_equal(g["sigma"].ravel(), sigma.astype(np.float32))
