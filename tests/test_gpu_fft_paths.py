"""De-dispersion and synthesis kernels at the branches of their transforms,
against the FP64 oracle: bands whose highest bin selects 4, 5, 6 or 8 rows of
the synthesis transform's first pass (both sides of each limit), one hop and
several, a single trial, a uniform grid (stepped chirp) and a non-uniform one.

Tolerance: a 4096-point transform and its inverse in FP32 have an error of
about sqrt(24 stages) 2^-24 = 3e-7 relative, and the FP32 phase of the chirp
(one rounding below 1/2 cycle, the hardware sine) adds about 5e-7: 2e-6 is
allowed.  The synthesis alone (10 stages, 16 taps) is allowed 1e-6."""
import numpy as np
import pytest

import oracle
from paper_1612_06592_amd import lp

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.sqrt(np.sum(np.abs(a - b) ** 2) / np.sum(np.abs(b) ** 2)))


def noise(rng, *shape):
    return (rng.standard_normal(shape + (2,)) * 50).astype(np.float32)


def cplx(a):
    return a[..., 0].astype(np.float64) + 1j * a[..., 1]


@pytest.mark.parametrize("k0,S", [(1, 3), (250, 6), (251, 5), (255, 2),
                                  (318, 2), (319, 1), (320, 1), (382, 2),
                                  (383, 2), (1, 511), (509, 3)])
@pytest.mark.parametrize("series", [False, True])
def test_synthesis_bands(k0, S, series):
    import torch
    n_t = 2048
    k = np.arange(k0, k0 + S, dtype=np.int32)
    rng = np.random.default_rng(k0 * 1000 + S)
    ns = 2
    d, hist = noise(rng, ns, S, n_t), noise(rng, ns, S, 16)
    ctx = lp.Ctx(0)
    dd, hh = (torch.from_numpy(a).to("cuda:0") for a in (d, hist))
    cand = torch.empty(lp.nbytes("lp_cand_bytes", ns, n_t), dtype=torch.uint8,
                       device="cuda:0")
    xo = torch.empty((ns, n_t * 1024), device="cuda:0") if series else None
    lp.synthesize(ctx, lp.Band(k), dd, ns, n_t, 4096, hh, cand, xo)
    torch.cuda.synchronize()
    past = np.ascontiguousarray(cplx(hist)[:, :, 1:].transpose(0, 2, 1))
    z = oracle.synthesize(oracle.prototype(), k, cplx(d), past)
    z = z.reshape(ns, n_t, 1024)
    head = cand[:ns * n_t * 8].view(torch.int32).view(ns, n_t, 2).cpu()
    emax = head[..., 0].contiguous().view(torch.float32).numpy()
    arg = head[..., 1].numpy()
    psum = cand[ns * n_t * 8:].view(torch.float32)[:ns * n_t // 16].cpu().numpy()
    env = 2 * np.abs(z)
    assert rel(emax, env.max(2)) <= 1e-6
    # The reported offset holds the maximum (to rounding, where two tie).
    at = np.take_along_axis(env, arg[..., None].astype(np.int64), 2)[..., 0]
    assert np.all(at >= env.max(2) * (1 - 1e-5))
    assert rel(psum, ((2 * z.real) ** 2).reshape(ns * n_t // 16, -1).sum(1)) <= 1e-6
    assert np.array_equal(hh.cpu().numpy(), d[:, :, -16:])
    if series:
        assert rel(xo.cpu().numpy().reshape(z.shape), 2 * z.real) <= 1e-6
    ctx.close()


@pytest.mark.parametrize("tec", [(7.0,), (0.0, 3.0), (2.0, 9.0, 16.0, 23.0),
                                 (1.0, 2.0, 30.0)])
@pytest.mark.parametrize("hops", [1, 2, 5])
def test_dedispersion_trials(tec, hops):
    import torch
    B, S, n_t = 2, 3, 2048 * hops
    k = np.array([40, 211, 400], dtype=np.int32)
    rng = np.random.default_rng(hops * 10 + len(tec))
    y, tail = noise(rng, B, S, n_t), noise(rng, B, S, 2048)
    ctx = lp.Ctx(0)
    yd, td = (torch.from_numpy(a).to("cuda:0") for a in (y, tail))
    d = torch.empty((B, len(tec), S, n_t, 2), device="cuda:0")
    lp.dedisperse(ctx, lp.Band(k), np.array(tec), yd, B, n_t, td, d)
    torch.cuda.synchronize()
    got = cplx(d.cpu().numpy())
    ref = oracle.dedisperse(k, np.array(tec), cplx(y), cplx(tail))
    assert rel(got, ref) <= 2e-6
    assert np.max(np.abs(got - ref)) <= 2e-5 * np.sqrt(np.mean(np.abs(ref) ** 2))
    assert np.array_equal(td.cpu().numpy(), y[:, :, -2048:])
    ctx.close()


@pytest.mark.parametrize("B,n_sb,hops", [(61, 68, 4), (23, 180, 4),
                                         (61, 30, 11)])
def test_dedispersion_runs_equal_single_hops(B, n_sb, hops):
    """Shapes large enough for the kernel that walks runs of hops (4 and more
    per workgroup, also where they do not divide the series): outputs and
    tail equal block-by-block calls of one hop each, which take the other
    kernel, bit for bit (a served stream's chunks may take either)."""
    import torch
    k = np.arange(60, 60 + n_sb, dtype=np.int32)
    g = torch.Generator(device="cuda:0").manual_seed(hops)
    n_t = 2048 * hops
    y = torch.randn((B, n_sb, n_t, 2), generator=g, device="cuda:0")
    t0 = torch.randn((B, n_sb, 2048, 2), generator=g, device="cuda:0")
    ctx, band, tec = lp.Ctx(0), lp.Band(k), np.array([11.0])
    d, tail = torch.empty_like(y), t0.clone()
    lp.dedisperse(ctx, band, tec, y, B, n_t, tail, d)
    ref, t1 = torch.empty_like(y), t0.clone()
    part = torch.empty((B, n_sb, 2048, 2), device="cuda:0")
    for h in range(hops):
        yh = y[:, :, 2048 * h:2048 * (h + 1)].contiguous()
        lp.dedisperse(ctx, band, tec, yh, B, 2048, t1, part)
        ref[:, :, 2048 * h:2048 * (h + 1)] = part
    assert torch.equal(tail, t1) and torch.equal(tail, y[:, :, -2048:])
    assert torch.equal(d, ref)
    ctx.close()
