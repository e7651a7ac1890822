"""The filterbank operators where many series share a call, which cuts each of
them into other runs of frames (one run of 416 frames here where one series
alone has runs of 32).

The solve of a series does not depend on the others: its vectors are the same
FP32 numbers, and its norms the same FP32 squares added in FP64, so x is equal
bit for bit and the norms to FP64's rounding over 2^17 terms in another order
(1e-13).  H and H^T against the FP64 oracle's operators, by runs of several
chunks and in several rounds of workgroups: within 1e-6, as for short runs."""
import numpy as np
import pytest

import oracle
from oracle import ppf_lsmr
from paper_1612_06592_amd import lp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nf", [(2, 500), (9, 2048), (48, 2063)])
def test_solve_does_not_depend_on_the_batch(ns, nf):
    import torch
    k, n_iter = np.arange(120, 160, dtype=np.int32), 7
    g = torch.Generator(device="cuda:0").manual_seed(nf)
    y = torch.randn((1, len(k), nf, 2), generator=g, device="cuda:0")
    ctx, band = lp.Ctx(0), lp.Band(k)

    def solve(y, ns):
        x = torch.full((ns, (nf - 15) * 1024), float("nan"), device="cuda:0")
        nb = lp.nbytes("lp_ppf_work_bytes", len(k), ns, nf)
        work = torch.full((nb // 4,), float("nan"), device="cuda:0")
        an = torch.zeros((ns, n_iter + 1), dtype=torch.float64, device="cuda:0")
        rn = torch.zeros(ns, dtype=torch.float64, device="cuda:0")
        lp.ppf_invert(ctx, band, y, ns, nf, n_iter, x, work.view(torch.uint8),
                      an, rn)
        return x, an, rn

    x1, an1, rn1 = solve(y, 1)
    x, an, rn = solve(y.expand(ns, -1, -1, -1).contiguous(), ns)
    for i in range(ns):
        assert torch.equal(x[i], x1[0])
    assert torch.max(torch.abs(an / an1 - 1)) <= 1e-13
    assert torch.max(torch.abs(rn / rn1 - 1)) <= 1e-13
    ctx.close()


@pytest.mark.parametrize("ns,nf", [(40, 500), (48, 2063), (900, 288)])
def test_long_runs_against_oracle(ns, nf):
    import torch
    k = np.array([3, 200, 511], dtype=np.int32)
    g = torch.Generator(device="cuda:0").manual_seed(nf)
    x = torch.randn((ns, (nf - 15) * 1024), generator=g, device="cuda:0")
    y = torch.randn((ns, 3, nf, 2), generator=g, device="cuda:0")
    ctx, band = lp.Ctx(0), lp.Band(k)
    hx, hty = torch.empty_like(y), torch.empty_like(x)
    lp.ppf_analyze(ctx, band, x, ns, nf, hx)
    lp.ppf_adjoint(ctx, band, y, ns, nf, hty)
    torch.cuda.synchronize()
    h = oracle.prototype()
    for i in (0, ns - 1):
        a = ppf_lsmr.analysis(h, 1024, k, x[i].cpu().numpy().astype(np.float64))
        b = hx[i].cpu().numpy().astype(np.float64)
        assert np.linalg.norm(b[..., 0] + 1j * b[..., 1] - a) <= 1e-6 * np.linalg.norm(a)
        yi = y[i].cpu().numpy().astype(np.float64)
        c = ppf_lsmr.adjoint(h, 1024, k, yi[..., 0] + 1j * yi[..., 1])
        d = hty[i].cpu().numpy().astype(np.float64)
        assert np.linalg.norm(d - c) <= 1e-6 * np.linalg.norm(c)
    ctx.close()
