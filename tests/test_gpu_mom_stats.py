"""The statistics pass of the median of MAD at W 4096, which takes half of a
window's samples into a histogram and counts the rest around the result:
signals for which that succeeds, misses, or lies at the ends of the range;
medians and MADs bit-exact against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1710_08576_amd as rfi
from paper_1710_08576_amd import synth

pytestmark = pytest.mark.gpu


def _signals(rng, n):
    g = lambda mu, sd: np.clip(np.round(rng.normal(mu, sd, n)), -128, 127)
    half = np.arange(n) % 16 < 8  # what the histogram sees
    step = g(0, 10)
    step[n // 4:] += 25
    return [g(0, 6), g(-3, 20), g(40, 1), g(0, 0.4), g(0, 60), g(120, 5), g(-126, 4), np.full(n, -7), np.full(n, 127),
            rng.integers(-128, 128, n), np.where(rng.random(n) < 0.5, -50, 50), np.where(half, 0, g(30, 10)),
            np.where(half, g(0, 3), g(0, 40)), np.where(rng.random(n) < 0.5, g(0, 30), 2), np.clip(step, -128, 127),
            np.where(half, 5, 6), np.where(half, 5, 8), np.where(half, 5, 9)]


@pytest.mark.parametrize("mode", [rfi.ZERO, rfi.CLIP])
def test_w4096_statistics(gpu, mode):
    rng = np.random.default_rng(77)
    streams = [np.asarray(s).astype(np.int8) for s in _signals(rng, 4096 * 9)]
    x = synth.pack([torch.as_tensor(s) for s in streams])
    L, n = [len(s) for s in streams], len(streams)
    y, st = rfi.mom_filter(x.to(gpu), L, [4096] * n, [3.0] * n, [mode] * n, 4, seed=2)
    yo, sto = oracle.mom_filter_batch(x.numpy(), L, [4096] * n, [3.0] * n, [mode] * n, 4, seed=2)
    assert np.array_equal(rfi.stats_numpy(st), sto)
    assert np.array_equal(y.cpu().numpy(), yo)
