"""int8 windows held in registers (any length and start): the sizes at the
edges of the kernels' thread counts and chunks, several windows per
workgroup with a ragged last workgroup, and carried heads; bit-exact against
the CPU oracle."""
import numpy as np
import pytest
import torch

import paper_1710_08576_amd as rfi
from paper_1710_08576_amd import synth

from _helpers import check_against_oracle, gpu_run

pytestmark = pytest.mark.gpu


def _streams(rng, n):
    g = lambda sd: np.clip(np.round(rng.normal(0, sd, n)), -128, 127)
    return [np.asarray(s).astype(np.int8) for s in (
        g(9), g(40), rng.integers(-128, 128, n), np.full(n, 127), np.where(rng.random(n) < 0.6, 127, g(30)),
        np.where(rng.random(n) < 0.5, -128, 127), g(2))]


# 64 threads hold 4066 samples at any start, or 8162 in eight chunks each, 128
# threads 16354, 256 threads 32738; longer windows take the two-pass kernel
@pytest.mark.parametrize("W", [1, 5, 15, 16, 17, 100, 511, 1000, 4066, 4067, 4095, 8162, 8163, 9000, 16354, 16355, 16383,
                               32738, 32739])
@pytest.mark.parametrize("mode", [rfi.ZERO, rfi.CLIP, rfi.NOISE])
def test_window_sizes(gpu, W, mode):
    rng = np.random.default_rng(W + mode)
    streams = [s[:len(s) - i] for i, s in enumerate(_streams(rng, 3 * W + W // 2 + 40))]
    x = synth.pack([torch.as_tensor(s) for s in streams])
    k = (3.0, 0.5, 1.5)
    specs = [synth.StreamSpec(len(s), W, k[i % 3], mode, 1, 0, 1, 1) for i, s in enumerate(streams)]
    y, st = gpu_run(x, specs, 9, gpu)
    check_against_oracle(x, specs, 9, y, st)


@pytest.mark.parametrize("modes", [(0, 1), (0, 1, 2)])
def test_modes_share_a_workgroup(gpu, modes):
    """Short streams of several modes and windows, in place: the windows of
    one workgroup belong to different streams, some of them not noise."""
    rng = np.random.default_rng(8)
    streams = [_streams(rng, 1500 + 13 * i)[i % 7] for i in range(21)]
    x = synth.pack([torch.as_tensor(s) for s in streams])
    specs = [synth.StreamSpec(len(s), (700, 1000, 1499)[i % 3], 1.0, modes[i % len(modes)], 1, 0, 1, 1)
             for i, s in enumerate(streams)]
    y, st = gpu_run(x, specs, 4, gpu, inplace=True)
    check_against_oracle(x, specs, 4, y, st, check_padding=False)


@pytest.mark.parametrize("W,mode", [(700, 2), (5000, 1), (12000, 2)])
def test_mom_chunked_replacement(gpu, W, mode):
    """Median of MAD on windows that are no tile class (chunks of two
    windows, tails, items of several windows), against the definition."""
    import oracle
    rng = np.random.default_rng(W)
    streams = [_streams(rng, 6 * W + 333)[i] for i in (0, 1, 2, 4)]
    x = synth.pack([torch.as_tensor(s) for s in streams])
    L = [len(s) for s in streams]
    y, st = rfi.mom_filter(x.to(gpu), L, [W] * 4, [2.0] * 4, [mode] * 4, 3, seed=6)
    yo, sto = oracle.mom_filter_batch(x.numpy(), L, [W] * 4, [2.0] * 4, [mode] * 4, 3, seed=6)
    so = rfi.layout(L, [W] * 4)[0]
    for o, n in zip(so, L):
        assert np.array_equal(y.cpu().numpy()[o:o + n], yo[o:o + n])
    assert np.array_equal(rfi.stats_numpy(st), sto)
