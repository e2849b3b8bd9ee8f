"""The order in which LayerNorm adds a row up: a lane's own values, then lanes 32 apart, 16, 8, .. 1, in every form of the kernel.  Values of
2^25 and -2^25 that meet in the first step cancel exactly; in any later one the ones beside them have been rounded away already."""
import numpy as np
import pytest

from paper_2412_11272_amd import binding as wf

pytestmark = pytest.mark.gpu


# rows of one to eight pieces of 256 values (four to a lane), few and many of them (gain and shift early or late)
@pytest.mark.parametrize("M", [3, 2500])
@pytest.mark.parametrize("d", [256, 512, 768, 1024, 1280, 2048])
def test_far_lanes_meet_first(M, d):
    import torch
    big = 2.0 ** 25
    small = np.float32(0.7)
    x = np.full((M, d), small)
    lane = np.arange(M) % 32
    x[np.arange(M), 4 * lane] = big
    x[np.arange(M), 4 * (lane + 32)] = -big
    # a lane's remaining values are zero where a big one is, so that its own sum is exact as well
    for k in range(0, d, 256):
        for off in range(4):
            for half in (0, 32):
                c = k + 4 * (lane + half) + off
                keep = np.abs(x[np.arange(M), c]) == big
                x[np.arange(M), c] = np.where(keep, x[np.arange(M), c], 0.0)
    mean = x.astype(np.float64).sum(1, keepdims=True) / d
    var = ((x - mean) ** 2).mean(1, keepdims=True)
    ref = (x - mean) / np.sqrt(var + 1e-5)
    out = torch.empty((M, d), dtype=torch.float32, device="cuda")
    wf.op_layernorm(torch.from_numpy(x).cuda(), torch.ones(d, device="cuda"), torch.zeros(d, device="cuda"), out)
    rest = x == small
    got = out.cpu().numpy()[rest]
    # The sums of 0.7 are off by a few 2^-24, value - mean is 1 / 32 of the mean and the scale off by as much again: 1e-5.  What the big
    # values' rounding to multiples of 2 and 4 takes from a sum of 0.7 d changes it by 2e-2 and more.
    assert np.abs(got / ref[rest] - 1).max() <= 1e-4
