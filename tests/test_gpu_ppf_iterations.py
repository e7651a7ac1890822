"""lp_ppf_invert stopped after every small number of iterations, odd and even:
x is brought up to date after every second one and by the closing step, and
hbar_0 = x_0 = 0 are never stored.  Work and output start as NaN, so that
whatever is read before it is written shows.

Against the FP64 oracle's iterate: each of H and H^T is within 1e-6 (relative
RMS) of its FP64 value, an iteration applies both, and so few iterations do not
amplify it yet: 2e-6 per iteration."""
import numpy as np
import pytest

import oracle
from oracle import ppf_lsmr
from paper_1612_06592_amd import lp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_iter", [1, 2, 3, 4, 5, 6])
def test_every_iteration_count(n_iter):
    import torch
    ns, nf, k = 2, 80, np.arange(120, 160, dtype=np.int32)
    rng = np.random.default_rng(n_iter)
    y = rng.standard_normal((ns, len(k), nf, 2)).astype(np.float32)
    ctx, band = lp.Ctx(0), lp.Band(k)
    x = torch.full((ns, (nf - 15) * 1024), float("nan"), device="cuda:0")
    nb = lp.nbytes("lp_ppf_work_bytes", len(k), ns, nf)
    work = torch.full((nb // 4,), float("nan"), device="cuda:0")
    lp.ppf_invert(ctx, band, torch.from_numpy(y).to("cuda:0"), ns, nf, n_iter,
                  x, work.view(torch.uint8))
    torch.cuda.synchronize()
    got = x.cpu().numpy().astype(np.float64)
    h = oracle.prototype()
    for i in range(ns):
        want, _ = ppf_lsmr.invert(h, 1024, k, y[i, ..., 0] + 1j * y[i, ..., 1].astype(np.float64),
                                  n_iter)
        assert np.linalg.norm(got[i] - want) <= 2e-6 * n_iter * np.linalg.norm(want)
    ctx.close()


@pytest.mark.parametrize("ns", [9, 12, 20])
def test_streaming_of_the_vectors_does_not_show(ns):
    """Many equal series, so that 1, 2 or 3 of the vectors bypass the caches,
    against one series alone (none does).  The cut into runs differs, so the
    norms are summed in another order (1e-7 in each partial sum's FP32): 5
    iterates agree within 1e-5."""
    import torch
    nf, k, n_iter = 2048, np.arange(120, 160, dtype=np.int32), 5
    g = torch.Generator(device="cuda:0").manual_seed(ns)
    y = torch.randn((1, len(k), nf, 2), generator=g, device="cuda:0")
    ctx, band = lp.Ctx(0), lp.Band(k)

    def solve(y, ns):
        x = torch.full((ns, (nf - 15) * 1024), float("nan"), device="cuda:0")
        nb = lp.nbytes("lp_ppf_work_bytes", len(k), ns, nf)
        work = torch.full((nb // 4,), float("nan"), device="cuda:0")
        lp.ppf_invert(ctx, band, y, ns, nf, n_iter, x, work.view(torch.uint8))
        return x.double()

    one = solve(y, 1)[0]
    many = solve(y.expand(ns, -1, -1, -1).contiguous(), ns)
    for i in range(ns):
        assert torch.linalg.norm(many[i] - one) <= 1e-5 * torch.linalg.norm(one)
    ctx.close()
