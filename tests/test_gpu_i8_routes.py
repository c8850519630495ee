"""Which kernel takes the int8 windows that are no tiles: short ones, few or
many of each length, short and long ones in one batch; every route bit-exact
against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1710_08576_amd as rfi
from paper_1710_08576_amd import synth

from _helpers import SENTINEL, check_against_oracle, gpu_run, unpack

pytestmark = pytest.mark.gpu


def _batch(seed, windows, counts, modes):
    """A stream per entry: counts[i] windows of windows[i] samples, the last
    one 3 samples short."""
    rng = np.random.default_rng(seed)
    kinds = (lambda n: rng.normal(0, 9, n), lambda n: rng.integers(-128, 128, n), lambda n: rng.normal(90, 40, n),
             lambda n: np.where(rng.random(n) < 0.6, 127, rng.normal(0, 30, n)))
    lens = [w * c - (3 if w > 3 else 0) for w, c in zip(windows, counts)]
    xs = [np.clip(np.round(kinds[i % 4](n)), -128, 127).astype(np.int8) for i, n in enumerate(lens)]
    specs = [synth.StreamSpec(n, w, (3.0, 0.5, 1.5)[i % 3], modes[i % len(modes)], 1, 0, 1, 1)
             for i, (n, w) in enumerate(zip(lens, windows))]
    return synth.pack([torch.as_tensor(v) for v in xs]), specs


# either side of: short windows, 512 and 4096 windows of a launch, the longest
# window of 64 and 128 threads, windows that nearly fill 256
@pytest.mark.parametrize("modes", [(0, 1), (2,), (0, 1, 2)])
@pytest.mark.parametrize("W", [160, 161, 256, 257, 4066, 4067, 8162, 8163, 11000, 11001, 14000, 14001, 15000, 15001, 16354])
@pytest.mark.parametrize("count", [512, 513, 4096, 4097])
def test_window_counts(gpu, W, count, modes):
    x, specs = _batch(W + count, [W] * 3, [count // 3, count // 3, count - 2 * (count // 3)], modes)
    y, st = gpu_run(x, specs, 9, gpu)
    check_against_oracle(x, specs, 9, y, st)


# short windows beside longer ones, in the longer ones' launch and in their own
@pytest.mark.parametrize("modes", [(0, 1), (2, 1, 0)])
@pytest.mark.parametrize("shorts", [4095, 4096])
def test_short_and_long_windows(gpu, shorts, modes):
    x, specs = _batch(shorts, [5, 700, 1, 160, 6000, 100], [shorts - 2000, 40, 900, 1, 9, 1099], modes)
    y, st = gpu_run(x, specs, 9, gpu)
    check_against_oracle(x, specs, 9, y, st)
    L, W, K, M = unpack(specs)
    yo, sto = oracle.filter_batch(x.numpy(), L, W, K, M, seed=9)
    xd = x.to(gpu)
    stn = torch.zeros((len(sto), 4), dtype=torch.int32, device=gpu)
    yn = torch.full_like(xd, SENTINEL)
    rfi.mad_filter_noalloc(xd, L, W, K, M, seed=9, y=yn, stats=stn)
    check_against_oracle(x, specs, 9, yn.cpu().numpy(), rfi.stats_numpy(stn))
    if 2 not in modes:
        ys, sts = rfi.mad_filter_multi(xd, L, W, [K, [2.0] * len(L)], [M, M[::-1]], seed=9)
        for yy, s, k, m in zip(ys, sts, (K, [2.0] * len(L)), (M, M[::-1])):
            yo, sto = oracle.filter_batch(x.numpy(), L, W, k, m, seed=9)
            for o, n in zip(rfi.layout(L, W)[0], L):
                assert np.array_equal(yy.cpu().numpy()[o:o + n], yo[o:o + n])
            assert np.array_equal(rfi.stats_numpy(s), sto)


def test_statistics_of_short_windows(gpu):
    """The statistics pass of the median of MAD on short windows only, and on
    many of them beside longer ones."""
    for windows, counts in (([7, 100, 2], [900, 300, 50]), ([7, 1000, 33], [4000, 20, 500])):
        x, specs = _batch(4, windows, counts, (0, 1, 2))
        L, W, K, M = unpack(specs)
        y, st = rfi.mom_filter(x.to(gpu), L, W, K, M, 5, seed=6)
        yo, sto = oracle.mom_filter_batch(x.numpy(), L, W, K, M, 5, seed=6)
        for o, n in zip(rfi.layout(L, W)[0], L):
            assert np.array_equal(y.cpu().numpy()[o:o + n], yo[o:o + n])
        assert np.array_equal(rfi.stats_numpy(st), sto)


@pytest.mark.parametrize("W", [5000, 9000])
def test_noalloc_many_noise_windows(gpu, W):
    """More windows than take the kernels of few: without allocation they keep
    to kernels that need no private memory."""
    x, specs = _batch(W, [W] * 2, [2200, 2000], (2, 1))
    L, W, K, M = unpack(specs)
    xd = x.to(gpu)
    y = torch.full_like(xd, SENTINEL)
    rfi.mad_filter_noalloc(xd, L, W, K, M, seed=9, y=y)
    check_against_oracle(x, specs, 9, y.cpu().numpy(), None)


# ends of streams, launches that the plan takes: one where it saves a launch,
# the split ones where the ends are many, or long ones in noise mode
@pytest.mark.parametrize("n,low,W,modes,launches", [
    (60, 20_000, 4096, (1,), 1), (8, 30_000, 2048, (2, 0), 1), (60, 31_000, 16384, (2,), 2), (60, 31_000, 8192, (2,), 2),
    (1000, 20_000, 512, (1,), 2), (1000, 20_000, 512, (0, 1), 3), (1000, 18_000, 16384, (1,), 1)])
def test_ends_of_streams(gpu, n, low, W, modes, launches):
    rng = np.random.default_rng(n + W)
    xs = [np.clip(np.round(rng.normal(0, 9, low + 7 * (i % 9))), -128, 127).astype(np.int8) for i in range(n)]
    specs = [synth.StreamSpec(len(v), W, 2.0, modes[i % len(modes)], 1, 0, 1, 1) for i, v in enumerate(xs)]
    x = synth.pack([torch.as_tensor(v) for v in xs])
    plan = rfi.Plan(1, *unpack(specs))
    assert plan.info()["launches"] == launches
    plan.close()
    y, st = gpu_run(x, specs, 9, gpu)
    check_against_oracle(x, specs, 9, y, st)
