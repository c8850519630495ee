"""int16 windows held in registers (any length up to 16384, any start): the
sizes at the edges of the kernels' thread counts, and sample distributions
that send the selection through one-value slots, wider slots and the
full-range histogram; bit-exact against the CPU oracle."""
import numpy as np
import pytest
import torch

import paper_1710_08576_amd as rfi
from paper_1710_08576_amd import synth

from _helpers import check_against_oracle, gpu_run

pytestmark = pytest.mark.gpu


def _signals(rng, n):
    """Streams of n samples: narrow, moderate and wide noise, uniform,
    bimodal, saturated at either end, constant, bursts, a level step."""
    g = lambda mu, sd: np.clip(np.round(rng.normal(mu, sd, n)), -32768, 32767)
    burst = g(100, 400)
    hit = rng.random(n) < 0.02
    burst[hit] = np.clip(20000 * rng.standard_t(2, int(hit.sum())), -32768, 32767)
    step = g(0, 300)
    step[n // 3:] += 9000
    out = [g(-20000, 3), g(0, 400), g(5000, 900), g(-700, 2500), g(0, 12000), rng.integers(-32768, 32768, n),
           np.where(rng.random(n) < 0.5, -25000, 25000), g(32750, 40), g(-32760, 300), g(31000, 4000),
           np.where(rng.random(n) < 0.6, 32767, g(0, 9000)), np.full(n, -32768), np.full(n, 32767), burst, step]
    return [np.asarray(s).astype(np.int16) for s in out]


# 64 threads hold 2048 samples (2041 at any start), 128 4096, or 8192 in eight
# chunks each, 256 14336, 512 16384; 16385 takes the radix kernel
@pytest.mark.parametrize("W", [9, 500, 512, 1000, 2041, 2042, 2048, 2049, 4088, 4096, 4097, 8184, 8185, 8191, 9001, 14329, 14336, 14337, 16376,
                               16377, 16384, 16385])
@pytest.mark.parametrize("mode", [rfi.ZERO, rfi.CLIP, rfi.NOISE])
def test_window_sizes(gpu, W, mode):
    rng = np.random.default_rng(W * 3 + mode)
    streams = [s[:len(s) - i] for i, s in enumerate(_signals(rng, 2 * W + W // 2 + 30))]
    x = synth.pack([torch.as_tensor(s) for s in streams])
    k = (3.0, 0.5, 2.0)
    specs = [synth.StreamSpec(len(s), W, k[i % 3], mode, 1, 0, 1, 1, "i16") for i, s in enumerate(streams)]
    y, st = gpu_run(x, specs, 9, gpu)
    check_against_oracle(x, specs, 9, y, st)


@pytest.mark.parametrize("schedule", ["split", "split_persist", "fused", "per_stream", "one_launch", "one_launch_persist"])
def test_mixed_sizes_every_schedule(gpu, schedule):
    """Streams of every thread count, of the tile class and of the radix
    kernel in one batch, in place."""
    rng = np.random.default_rng(5)
    windows = [512, 1000, 3000, 4096, 7001, 8192, 16384, 16000, 20000, 2048]
    streams = [_signals(rng, 40000 + 17 * i)[i % 5 + 1] for i in range(len(windows))]
    x = synth.pack([torch.as_tensor(s) for s in streams])
    specs = [synth.StreamSpec(len(s), w, 2.5, i % 3, 1, 0, 1, 1, "i16") for i, (s, w) in enumerate(zip(streams, windows))]
    y, st = gpu_run(x, specs, 4, gpu, schedule=schedule, inplace=True)
    check_against_oracle(x, specs, 4, y, st, check_padding=False)
