"""ADC codes bit for bit against the oracle where the kernel branches: word
counts around whole groups of four and batches of four groups, sample ranges
that do not fill a workgroup's 1024 samples, and a counter that passes 2^32
inside a workgroup."""
import numpy as np
import pytest

from oracle import station_sim
from paper_1612_06592_amd import lp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [0, 1, 3, 4, 5, 15, 16, 17, 20, 33, 48])
@pytest.mark.parametrize("n0,n", [(0, 1), (5, 255), (2 ** 32 - 700, 1500),
                                  (2 ** 40 + 3, 1025)])
def test_codes(R, n0, n):
    import torch
    seed, n_in = 0x1234567_89ABCDEF + R, 3
    ctx = lp.Ctx(0)
    adc = torch.full((n_in, n + 64), 77, dtype=torch.int16, device="cuda:0")
    out = adc.view(-1)[:n_in * n]
    lp.sim_adc(ctx, seed, n_in, R, 12, n0, n, out)
    torch.cuda.synchronize()
    ref = station_sim.adc(seed, n_in, R, 12, n0, n)
    assert np.array_equal(out.cpu().numpy().reshape(n_in, n), ref)
    assert bool((adc.view(-1)[n_in * n:] == 77).all())
    ctx.close()
