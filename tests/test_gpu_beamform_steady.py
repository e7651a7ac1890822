"""Both beamformers where a workgroup walks several tiles (the next one loaded
while the present one is multiplied), against the FP64 oracle.

FP16: every kernel instance, by k-steps of 8 inputs, load width (rows that are
multiples of 16, 8 and 4 bytes) and one or two n-tiles to a wave; nine tiles of
128 rows or eighteen of 64, so that the last workgroup's walk ends early.  The
weights are rounded to FP16 (2^-11 relative), the samples are exact and the
sums FP32: below 2^-11 relative RMS, and no element off by 1e-2 of the RMS.

FP32: more pieces of rows than the chip has waves, for one and several n-tiles
and workgroups of four and eight waves; the first, a middle and the last subband
are compared.  2 K products with one rounding each: below 2e-6 relative RMS, and
no element off by 2e-5 of the RMS."""
import numpy as np
import pytest

import oracle
from paper_1612_06592_amd import lp

pytestmark = pytest.mark.gpu


def compare(rng, n_in, B, S, n_t, dtype, prec, gains, rms_tol, max_tol):
    import torch
    enu = np.stack([rng.uniform(-900, 900, n_in), rng.uniform(-900, 900, n_in),
                    np.zeros(n_in)], 1)
    azel = np.stack([rng.uniform(0, 6, B), rng.uniform(0.4, 1.2, B)], 1)
    gain = rng.uniform(0.2, 5, n_in).astype(np.float32) if gains else None
    k = np.arange(100, 100 + S, dtype=np.int32)
    lim = 127 if dtype == "ci8" else 2048
    xd = torch.randint(-lim, lim + 1, (S, n_t, n_in, 2), device="cuda:0",
                       dtype=torch.int8 if dtype == "ci8" else torch.int16,
                       generator=torch.Generator("cuda:0").manual_seed(n_in))
    y = torch.full((B, S, n_t, 2), float("nan"), device="cuda:0")
    ctx = lp.Ctx(0)
    lp.beamform(ctx, lp.Array(enu, 1, gain), lp.Band(k), lp.Dirs(azel), xd,
                n_t, lp.LP_CI8 if dtype == "ci8" else lp.LP_CI16, prec, y)
    torch.cuda.synchronize()
    ctx.close()
    some = sorted({0, S // 2, S - 1})
    ref = oracle.beamform(enu, 1, k[some], azel, xd[some].cpu().numpy(),
                          gain=gain)
    got = y[:, some].cpu().numpy().astype(np.float64)
    off = got[..., 0] + 1j * got[..., 1] - ref
    rms = np.sqrt(np.mean(np.abs(ref) ** 2))
    assert np.sqrt(np.mean(np.abs(off) ** 2)) <= rms_tol * rms
    assert np.max(np.abs(off)) <= max_tol * rms
    assert bool(torch.isfinite(y).all())


FP16 = [(8 * ks - less, "ci8") for ks in range(1, 17) for less in (0, 4, 6)]
FP16 += [(8 * ks - less, "ci16") for ks in range(1, 9) for less in (0, 2, 7)]


@pytest.mark.parametrize("n_in,dtype", FP16)
def test_fp16_instances(n_in, dtype):
    rng = np.random.default_rng(n_in)
    for B in ([3, 25], [16, 33], [8, 17], [9, 64])[n_in // 2 % 4]:
        compare(rng, n_in, B, 2, 1024 + 128, dtype, lp.LP_FP16_MFMA,
                n_in % 3 == 0, 2.0 ** -11, 1e-2)


@pytest.mark.parametrize("n_in,B,S,n_t,dtype", [
    (8, 1, 100, 16384, "ci16"), (8, 1, 100, 16384, "ci8"),
    (24, 17, 100, 4096, "ci16"), (40, 9, 99, 4096, "ci8"),
    (96, 37, 100, 4096, "ci16"), (96, 61, 100, 4096, "ci16"),
    (97, 8, 70, 4096, "ci16"), (128, 64, 40, 8192, "ci8")])
def test_fp32_walks(n_in, B, S, n_t, dtype):
    compare(np.random.default_rng(n_in * 100 + B), n_in, B, S, n_t, dtype,
            lp.LP_FP32, False, 2e-6, 2e-5)
