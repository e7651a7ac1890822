"""Results over 256 MB, which the de-dispersion and the second beamforming stage
write past the cache: the same bits as the same beams in smaller calls, which
leave theirs in it."""
import numpy as np
import pytest

from paper_1612_06592_amd import lp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tec", [(0.0, 3.0, 6.0), (1.0, 2.0, 30.0)])
def test_dedispersion_trials(tec):
    import torch
    B, n_sb, hops, J = 8, 100, 7, len(tec)
    n_t = 2048 * hops
    assert B * J * n_sb * n_t * 8 > 256 << 20 > 4 * J * n_sb * n_t * 8
    k = np.arange(80, 80 + n_sb, dtype=np.int32)
    g = torch.Generator(device="cuda:0").manual_seed(J)
    y = torch.randn((B, n_sb, n_t, 2), generator=g, device="cuda:0")
    t0 = torch.randn((B, n_sb, 2048, 2), generator=g, device="cuda:0")
    ctx, band = lp.Ctx(0), lp.Band(k)

    def run(y, t):
        d = torch.empty((len(y), J, n_sb, n_t, 2), device="cuda:0")
        t = t.clone()
        lp.dedisperse(ctx, band, np.array(tec), y, len(y), n_t, t, d)
        return d, t

    d, t = run(y, t0)
    for a in (0, 4):
        dp, tp = run(y[a:a + 4].clone(), t0[a:a + 4])
        assert torch.equal(d[a:a + 4], dp) and torch.equal(t[a:a + 4], tp)
    ctx.close()


@pytest.mark.parametrize("n_t,G", [(8192, 8), (8191, 8), (8192, 9)])
def test_second_stage(n_t, G):
    import torch
    n_st, n_sb, B, P = 18, 70, 61, 3
    assert B * n_sb * n_t * 8 > 256 << 20 > 20 * n_sb * n_t * 8
    rng = np.random.default_rng(n_t + G)
    enu = np.ascontiguousarray(rng.uniform(-1500, 1500, (n_st, 3)))
    azel = np.array([2.0, 0.8]) + rng.uniform(-0.01, 0.01, (B, 2))
    ctx, array = lp.Ctx(0), lp.Array(enu, 2)
    band = lp.Band(np.arange(80, 80 + n_sb, dtype=np.int32))
    groups = lp.Groups(np.arange(n_st) % G, G)
    prelim = lp.Dirs(np.ascontiguousarray(azel[:P]))
    g = torch.Generator(device="cuda:0").manual_seed(G)
    y1 = torch.randn((G * P, n_sb, n_t, 2), generator=g, device="cuda:0")

    def run(a, b):
        y = torch.empty((b - a, n_sb, n_t, 2), device="cuda:0")
        lp.beamform_stage2(ctx, array, groups, band, prelim,
                           lp.Dirs(np.ascontiguousarray(azel[a:b])), y1, n_t, y)
        return y

    y = run(0, B)
    for a, b in ((0, 20), (41, 61)):
        assert torch.equal(y[a:b], run(a, b))
    ctx.close()
