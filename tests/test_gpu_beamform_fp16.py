"""The FP16 beamformer's kernel instances (k-steps of 8 inputs, load widths of
4, 8 and 16 bytes, one to eight n-tiles of 8 beams), with and without input
gains, against the FP64 oracle.

Tolerance: the samples are exact in FP16 (|x| <= 2048) and the products
accumulate in FP32; the weights are rounded to FP16, at most 2^-11 relative,
so the outputs' relative RMS error is below 2^-11 = 4.9e-4.  No element is
off by more than 1e-2 of the RMS."""
import numpy as np
import pytest

import oracle
from paper_1612_06592_amd import lp

pytestmark = pytest.mark.gpu

CASES = [(n, "ci8") for n in (2, 6, 8, 12, 16, 18, 24, 28, 32, 40, 46, 48, 56,
                              64, 66, 72, 76, 80, 88, 96, 104, 112, 120, 128)]
CASES += [(n, "ci16") for n in (1, 3, 4, 8, 10, 12, 16, 20, 24, 31, 32, 36, 44,
                                48, 56, 60, 64)]


@pytest.mark.parametrize("n_in,dtype", CASES)
def test_instances_against_oracle(n_in, dtype):
    import torch
    rng = np.random.default_rng(n_in)
    S, n_t = 2, 128 * (1 + n_in % 3)
    beams = [1, 8, 9, 17, 24, 25, 33, 64]
    k = np.array([77, 300], dtype=np.int32)
    enu = np.stack([rng.uniform(-900, 900, n_in), rng.uniform(-900, 900, n_in),
                    np.zeros(n_in)], 1)
    lim = 127 if dtype == "ci8" else 2048
    x = rng.integers(-lim, lim + 1, (S, n_t, n_in, 2)).astype(
        np.int8 if dtype == "ci8" else np.int16)
    ctx, xd = lp.Ctx(0), torch.from_numpy(x).to("cuda:0")
    for B, gains in [(beams[n_in % 8], False), (beams[(n_in + 3) % 8], True)]:
        azel = np.stack([rng.uniform(0, 6, B), rng.uniform(0.4, 1.2, B)], 1)
        gain = rng.uniform(0.2, 5, n_in).astype(np.float32) if gains else None
        y = torch.full((B, S, n_t, 2), float("nan"), device="cuda:0")
        lp.beamform(ctx, lp.Array(enu, 1, gain), lp.Band(k), lp.Dirs(azel), xd,
                    n_t, lp.LP_CI8 if dtype == "ci8" else lp.LP_CI16,
                    lp.LP_FP16_MFMA, y)
        got = y.cpu().numpy().astype(np.float64)
        got = got[..., 0] + 1j * got[..., 1]
        ref = oracle.beamform(enu, 1, k, azel, x, gain=gain)
        rms = np.sqrt(np.mean(np.abs(ref) ** 2))
        assert np.sqrt(np.mean(np.abs(got - ref) ** 2)) <= 2.0 ** -11 * rms
        assert np.max(np.abs(got - ref)) <= 1e-2 * rms
    ctx.close()
