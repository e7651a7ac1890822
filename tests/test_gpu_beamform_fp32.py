"""The FP32 beamformer on the matrix cores at the edges of its tiles, against
the FP64 oracle: inputs around the k-groups of 8 inputs and the kernel
instances, rows of every load width (4, 8 and 16 bytes) and rows that no wide
load divides, beams around the 8-beam n-tiles, one and many pieces of 32 or 64
rows, and workgroup ranges that cross subbands.

Tolerance: an output is a sum of 2 K products of weights rounded to FP32
(2^-24) with one rounding per term, so its error is below about sqrt(2 K)
2^-24 relative: 1e-6 for K = 128; 2e-6 is allowed.  No element may be off by
more than 2e-5 of the output's RMS (a lost or doubled sample is of the order
of the RMS)."""
import numpy as np
import pytest

import oracle
from paper_1612_06592_amd import lp

pytestmark = pytest.mark.gpu

CASES = [  # n_in, beams, subbands, n_t, dtype
    (1, 1, 3, 128, "ci16"), (2, 1, 2, 256, "ci8"), (3, 5, 2, 128, "ci16"),
    (8, 8, 5, 384, "ci16"), (9, 9, 3, 128, "ci16"), (16, 7, 2, 1152, "ci8"),
    (18, 9, 3, 128, "ci8"), (20, 8, 4, 256, "ci16"), (25, 3, 2, 128, "ci16"),
    (32, 16, 2, 640, "ci8"), (33, 17, 2, 128, "ci16"), (48, 1, 7, 512, "ci8"),
    (56, 24, 2, 128, "ci8"), (64, 61, 3, 256, "ci16"), (66, 2, 2, 128, "ci8"),
    (72, 19, 2, 384, "ci8"), (80, 33, 2, 128, "ci16"),
    (96, 61, 40, 128, "ci16"), (96, 37, 3, 2048, "ci16"),
    (112, 64, 2, 128, "ci8"), (127, 5, 2, 128, "ci16"),
    (128, 64, 3, 256, "ci16"),
]


@pytest.mark.parametrize("n_in,B,S,n_t,dtype", CASES)
def test_tiles_against_oracle(n_in, B, S, n_t, dtype):
    import torch
    rng = np.random.default_rng(n_in * 1000 + B)
    enu = np.stack([rng.uniform(-900, 900, n_in), rng.uniform(-900, 900, n_in),
                    np.zeros(n_in)], 1)
    azel = np.stack([rng.uniform(0, 6, B), rng.uniform(0.4, 1.2, B)], 1)
    k = np.arange(100, 100 + S, dtype=np.int32)
    lim = 127 if dtype == "ci8" else 32767
    x = rng.integers(-lim, lim + 1, (S, n_t, n_in, 2)).astype(
        np.int8 if dtype == "ci8" else np.int16)
    ref = oracle.beamform(enu, 1, k, azel, x)
    ctx = lp.Ctx(0)
    y = torch.full((B, S, n_t, 2), float("nan"), device="cuda:0")
    lp.beamform(ctx, lp.Array(enu, 1), lp.Band(k), lp.Dirs(azel),
                torch.from_numpy(x).to("cuda:0"), n_t,
                lp.LP_CI8 if dtype == "ci8" else lp.LP_CI16, lp.LP_FP32, y)
    torch.cuda.synchronize()
    got = y.cpu().numpy().astype(np.float64)
    got = got[..., 0] + 1j * got[..., 1]
    ctx.close()
    rms = np.sqrt(np.mean(np.abs(ref) ** 2))
    assert np.sqrt(np.mean(np.abs(got - ref) ** 2)) <= 2e-6 * rms
    assert np.max(np.abs(got - ref)) <= 2e-5 * rms
