"""Median of MAD over the whole range of its arguments, bit-exact against the
CPU oracle: windows longer than a 16 KiB tile."""
import numpy as np
import pytest
import torch

import oracle
import paper_1710_08576_amd as rfi
from paper_1710_08576_amd import synth

pytestmark = pytest.mark.gpu


def _compare(y, st, x, L, W, K, M, mom_k, seed):
    yo, sto = oracle.mom_filter_batch(x, L, W, K, M, mom_k, seed=seed)
    for s, (o, n) in enumerate(zip(rfi.layout(L, W)[0], L)):
        assert np.array_equal(y[o:o + n], yo[o:o + n]), s
    assert np.array_equal(st, sto)


@pytest.mark.parametrize("W", [16400, 20000, 24576, 32768, 65536])
@pytest.mark.parametrize("mode", [rfi.ZERO, rfi.CLIP, rfi.NOISE])
def test_windows_above_a_tile(gpu, W, mode):
    """Streams that end with a window of exactly 16384 samples, of one less,
    and with a whole window."""
    L = [16384, W + 16384, W + 16383, 2 * W]
    specs = [synth.StreamSpec(n, W, 2.0, mode, 9.0, 0.01, 8, 3000) for n in L]
    x = synth.gen_packed(specs, W + mode, 31)
    args = (L, [W] * 4, [2.0] * 4, [mode] * 4, 2)
    y, st = rfi.mom_filter(x.to(gpu), *args, seed=5)
    _compare(y.cpu().numpy(), rfi.stats_numpy(st), x.numpy(), *args, 5)
