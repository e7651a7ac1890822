"""The FP32 beamformer around the rule that sends few inputs or few beams to the
vector ALUs, and where an instance for more inputs or narrower loads is taken:
1 to 8 inputs at 1 beam to more than the rule's product, 9 to 28 inputs at one to
three beams, rows of every load width, half-filled and whole tiles of 256 rows.

Against the FP64 oracle: 2 K products of weights rounded to FP32, one rounding
each, below 2e-6 relative RMS and no element off by 2e-5 of the RMS.  And a call
equals the calls of its parts bit for bit: no route depends on the length."""
import numpy as np
import pytest

import oracle
from paper_1612_06592_amd import lp

pytestmark = pytest.mark.gpu

CASES = [(n, B, d) for n in (2, 4, 6, 8) for B in (1, 4, 25, 26, 51) for d in ("ci8", "ci16")]
CASES += [(n, B, "ci16") for n in (1, 3) for B in (1, 33, 34, 64)]
CASES += [(n, B, d) for n in (10, 12, 14, 16, 18, 20, 24, 26, 28, 30)
          for B in (1, 2, 3) for d in ("ci8", "ci16")]
CASES += [(n, B, "ci16") for n in (9, 11, 21, 27, 29) for B in (1, 2)]
CASES += [(n, B, "ci8") for n in (28, 36, 40, 50, 56, 72, 88, 104) for B in (1, 8, 9)]


@pytest.mark.parametrize("n_in,B,dtype", CASES)
def test_routes(n_in, B, dtype):
    import torch
    rng = np.random.default_rng(100 * n_in + B)
    S, n_t = 2, 128 * (1 + 2 * (B % 3))
    enu = np.stack([rng.uniform(-900, 900, n_in), rng.uniform(-900, 900, n_in),
                    np.zeros(n_in)], 1)
    azel = np.stack([rng.uniform(0, 6, B), rng.uniform(0.4, 1.2, B)], 1)
    k = np.array([77, 300], dtype=np.int32)
    lim = 127 if dtype == "ci8" else 32767
    x = rng.integers(-lim, lim + 1, (S, n_t, n_in, 2)).astype(
        np.int8 if dtype == "ci8" else np.int16)
    ctx, array, band, dirs = lp.Ctx(0), lp.Array(enu, 1), lp.Band(k), lp.Dirs(azel)

    def run(x):
        y = torch.full((B, S, x.shape[1], 2), float("nan"), device="cuda:0")
        lp.beamform(ctx, array, band, dirs, torch.from_numpy(x).to("cuda:0"),
                    x.shape[1], lp.LP_CI8 if dtype == "ci8" else lp.LP_CI16,
                    lp.LP_FP32, y)
        return y

    y = run(x)
    for t in range(0, n_t, 128):
        assert torch.equal(y[:, :, t:t + 128],
                           run(np.ascontiguousarray(x[:, t:t + 128])))
    got = y.cpu().numpy().astype(np.float64)
    ref = oracle.beamform(enu, 1, k, azel, x)
    off = got[..., 0] + 1j * got[..., 1] - ref
    ctx.close()
    rms = np.sqrt(np.mean(np.abs(ref) ** 2))
    assert np.sqrt(np.mean(np.abs(off) ** 2)) <= 2e-6 * rms
    assert np.max(np.abs(off)) <= 2e-5 * rms
