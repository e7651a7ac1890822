"""The trigger's launch paths against the oracle's rules, exactly: one or
several beams, one or several trials (each combination runs other kernels),
more beams than one scan holds, and lengths around a pass's 16384 windows."""
import numpy as np
import pytest

import oracle
from test_gpu_trigger import check_equal, make_cand, run_gpu_trigger
from paper_1612_06592_amd import lp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_beams,n_tec,n_t", [
    (1, 1, 2048), (1, 1, 16384), (1, 1, 18432), (1, 1, 65536), (3, 1, 4096),
    (1, 5, 2048), (4, 3, 2048), (1, 130, 2048), (1024, 1, 2048),
    (1025, 1, 2048), (1100, 2, 2048)])
@pytest.mark.parametrize("frame0", [0, 5000])
def test_paths_equal_oracle(n_beams, n_tec, n_t, frame0):
    rng = np.random.default_rng(n_beams * 100 + n_tec)
    ns, k_sigma = n_beams * n_tec, 2.0 + 1.0 / 512
    raw, sigma, wmax, warg = make_cand(
        rng, n_beams, n_tec, n_t, frame0, rng.integers(-2, 4, ns), 0.01,
        k_sigma)
    trig, snr, best = oracle.trigger(sigma, wmax, warg, n_beams, n_tec, n_t,
                                     frame0, lp.WARM_FRAMES, k_sigma)
    for cap in (len(trig) + 10, max(1, len(trig) // 2)):
        g = run_gpu_trigger(raw, n_beams, n_tec, n_t, frame0, k_sigma, cap)
        check_equal(g, trig, cap)
        assert np.array_equal(g["snr"], snr.astype(np.float32))
        assert np.array_equal(g["best"], best)
        assert np.array_equal(g["sigma"].ravel(), sigma.astype(np.float32))
