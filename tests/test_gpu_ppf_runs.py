"""H and H^T over every way that a series is cut into workgroups' runs: lengths
around the 32-frame chunks and the runs' ends, several series, sizes up to one
round of workgroups (several rounds and longer runs: test_gpu_ppf_batch.py).

The cut must not show: the same frames inside a longer series and inside many
series (other runs) give the same bits.  And against the FP64 oracle's
operators: 16 taps and ten transform stages in FP32 are within 1e-6."""
import numpy as np
import pytest

from oracle import ppf_lsmr
import oracle
from paper_1612_06592_amd import lp

pytestmark = pytest.mark.gpu


def operators(ctx, band, x, y, ns, nf):
    import torch
    hx = torch.empty_like(y)
    hty = torch.empty_like(x)
    lp.ppf_analyze(ctx, band, x, ns, nf, hx)
    lp.ppf_adjoint(ctx, band, y, ns, nf, hty)
    return hx, hty


@pytest.mark.parametrize("nf", [16, 17, 31, 32, 33, 47, 48, 63, 64, 65, 143,
                                144, 145, 271, 288, 500])
def test_run_ends_against_oracle(nf):
    import torch
    k = np.array([3, 200, 511], dtype=np.int32)
    ns = 2
    g = torch.Generator(device="cuda:0").manual_seed(nf)
    x = torch.randn((ns, (nf - 15) * 1024), generator=g, device="cuda:0")
    y = torch.randn((ns, 3, nf, 2), generator=g, device="cuda:0")
    ctx = lp.Ctx(0)
    hx, hty = operators(ctx, lp.Band(k), x, y, ns, nf)
    torch.cuda.synchronize()
    h = oracle.prototype()
    for i in range(ns):
        a = ppf_lsmr.analysis(h, 1024, k, x[i].cpu().numpy().astype(np.float64))
        b = hx[i].cpu().numpy().astype(np.float64)
        b = b[..., 0] + 1j * b[..., 1]
        assert np.linalg.norm(b - a) <= 1e-6 * np.linalg.norm(a)
        yi = y[i].cpu().numpy().astype(np.float64)
        c = ppf_lsmr.adjoint(h, 1024, k, yi[..., 0] + 1j * yi[..., 1])
        d = hty[i].cpu().numpy().astype(np.float64)
        assert np.linalg.norm(d - c) <= 1e-6 * np.linalg.norm(c)
    ctx.close()


@pytest.mark.parametrize("nf,many", [(1000, 40), (9000, 3), (20000, 2)])
def test_runs_do_not_show(nf, many):
    import torch
    k = np.arange(90, 100, dtype=np.int32)
    g = torch.Generator(device="cuda:0").manual_seed(nf)
    x = torch.randn((many, (nf - 15) * 1024), generator=g, device="cuda:0")
    y = torch.randn((many, 10, nf, 2), generator=g, device="cuda:0")
    ctx, band = lp.Ctx(0), lp.Band(k)
    hx, hty = operators(ctx, band, x, y, many, nf)
    for i in (0, many - 1):
        a, b = operators(ctx, band, x[i:i + 1].clone(), y[i:i + 1].clone(), 1,
                         nf)
        assert torch.equal(a[0], hx[i]) and torch.equal(b[0], hty[i])
    ctx.close()
