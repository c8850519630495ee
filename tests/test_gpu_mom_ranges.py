"""Median of MAD over the whole range of its arguments, bit-exact against the
CPU oracle: windows longer than a 16 KiB tile, and noise from any absolute
index."""
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


@pytest.mark.parametrize("W", [512, 4096, 16384, 1000])
@pytest.mark.parametrize("base", [0, 1, 2, 3, 4097])
def test_noise_at_any_absolute_index(gpu, W, base):
    """A stream whose first sample has an absolute index that is no multiple
    of 4: sample j of whole tiles and of tails draws word j & 3 of block
    j >> 2 (mom_k 1, so each window equals the plain filter's)."""
    L, k, seed = 2 * 16384 + 700, 1.5, 11
    x = synth.gen_packed([synth.StreamSpec(L, W, k, rfi.NOISE, 9.0, 0.01, 8, 3000)], W + base, 31)
    absb = torch.tensor([base], dtype=torch.int64, device=gpu)
    y, st = rfi.mom_filter_carry(x.to(gpu), [L], [W], [k], [rfi.NOISE], 1, absb, None, None, seed=seed)
    y, st, xn = y.cpu().numpy(), rfi.stats_numpy(st), x.numpy()
    for w, o in enumerate(range(0, L, W)):
        n = min(W, L - o)
        yo, so = oracle.window(xn[o:o + n], k, rfi.NOISE, abs_start=base + o, stream=0, seed=seed)
        assert np.array_equal(y[o:o + n], yo), w
        assert st[w] == so, w
