"""The work that a user of this library has it do, as measurable cases.

A case is a dict of plain values; `listed()` names the fixed ones, `draw()`
gives more of the same ranges, `prepare()` builds what a program holds before
the call (samples on the GPU, output buffers, the per-stream settings, a
server), `run()` makes one pass through the public entry points, `work()`
states what a pass cannot do without and `exact()` computes the results of a
pass in 64-bit integers and floats without the library.

Kinds of case:

  filter    mad_filter on an int8 or int16 batch of packed streams
  multi     mad_filter_multi: three outputs of one int8 input
  mom       mom_filter: threshold from the median of the last mom_k MADs
  carry     mom_filter_carry: the same on streams that arrive in pieces
  power     block_power of an input and of its filtered form + improvement
  serve     Server.replay_ptrs: one block of every stream, all ready at once

Sizes are per stream ("samples"); with "ragged" the streams' lengths are
spread over [1/2, 1] of it.  "window" 0 and "mode" "mixed" give every stream
its own (windows from the six tile classes).  "layout" seeds these choices,
so that a case has the same sizes whatever the inputs' seed.
"""
import random

import numpy as np
import torch

import paper_1710_08576_amd as rfi
from paper_1710_08576_amd import _lib, synth

CLASSES = (512, 1024, 2048, 4096, 8192, 16384)
MODES = {"zero": 0, "clip": 1, "noise": 2}
NOISE_SEED = 7
SEGMENT = 4  # blocks per segment of the improvement metric


def _case(name, kind, dtype, streams, samples, window, mode, ragged=False, mom_k=1, block=0, layout=1):
    c = {"kind": kind, "dtype": dtype, "streams": streams, "samples": samples, "window": window, "mode": mode,
         "ragged": ragged, "mom_k": mom_k, "block": block, "layout": layout}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # One antenna's short capture with a short last window, looked at by
        # hand: the call's own cost.
        _case("i8_one_short_stream", "filter", "i8", 1, 20000, 4096, "clip"),
        # The real-time backend: one block of 10^6 samples of each of 60
        # streams (30 antennas x 2 polarisations) is ready; windows of
        # 1024..16384 differ by stream and do not divide the block, so every
        # block starts with carried samples.
        _case("serve_60_blocks", "serve", "i8", 60, 1000000, 0, "clip"),
        # The headline batch: 60 long streams, digital-noise replacement.
        _case("i8_scale_w4096_noise", "filter", "i8", 60, 1 << 24, 4096, "noise"),
        # The narrowest window class, for short RFI, zeroing.
        _case("i8_w512_zero", "filter", "i8", 60, 1 << 22, 512, "zero"),
        # A window that is set in time, not in a power of two of samples.
        _case("i8_w5000_noise", "filter", "i8", 60, 1 << 22, 5000, "noise"),
        # An observation's batch of uneven streams, each with its own
        # window, threshold and replacement.
        _case("i8_mixed_batch", "filter", "i8", 64, 1 << 23, 0, "mixed", ragged=True),
        # 16-bit baseband at the usual window.
        _case("i16_w8192_noise", "filter", "i16", 60, 1 << 23, 8192, "noise"),
        # 16-bit baseband at the int8 filter's window.
        _case("i16_w4096_clip", "filter", "i16", 60, 1 << 21, 4096, "clip", ragged=True),
        # Side-by-side test of thresholds and replacements on one input.
        _case("multi_three_outputs", "multi", "i8", 60, 1 << 22, 4096, "zero"),
        # Median of MAD over the paper's history of 4096 windows.
        _case("mom_w4096_k4096", "mom", "i8", 60, 1 << 23, 4096, "zero", mom_k=4096),
        # The same in real time: one block of each stream with its history.
        _case("mom_carry_blocks", "carry", "i8", 60, 1 << 20, 4096, "noise", mom_k=4096),
        # Scoring a filter's output: integrated power before and after.
        _case("power_improvement", "power", "i8", 60, 1 << 23, 0, "zero", block=1 << 18),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _window(rng):
    return rng.choice(CLASSES) if rng.random() < 0.6 else _log_uniform(rng, 512, 16384)


def draw(rng):
    kind = rng.choice(["filter"] * 6 + ["multi", "mom", "carry", "power", "serve"])
    layout = rng.randrange(1 << 16)
    mode = rng.choice(["zero", "clip", "noise"])
    streams = rng.randint(1, 64)
    if kind == "filter":
        dtype = rng.choice(["i8", "i8", "i16"])
        total = _log_uniform(rng, 1 << 14, 1 << 26 if dtype == "i16" else 1 << 28)
        streams = min(streams, max(1, total >> 13))
        mixed = rng.random() < 0.25
        return _case(None, kind, dtype, streams, max(1, total // streams), 0 if mixed else _window(rng),
                     "mixed" if mixed else mode, ragged=rng.random() < 0.5, layout=layout)
    if kind == "serve":
        return _case(None, kind, "i8", streams, 16 * _log_uniform(rng, 1 << 12, 1 << 16), 0, mode, layout=layout)
    if kind == "power":
        return _case(None, kind, rng.choice(["i8", "i16"]), streams, _log_uniform(rng, 1 << 18, 1 << 21), 0, mode,
                     ragged=rng.random() < 0.5, block=_log_uniform(rng, 1 << 12, 1 << 16), layout=layout)
    samples = _log_uniform(rng, 1 << 16, 1 << 21)
    mom_k = _log_uniform(rng, 4, 4096) if kind in ("mom", "carry") else 1
    return _case(None, kind, "i8", streams, samples, _window(rng), mode, ragged=rng.random() < 0.5, mom_k=mom_k,
                 layout=layout)


# ---------------------------------------------------------------------------
# What a case fixes whatever its inputs: lengths, windows, thresholds, modes.
# ---------------------------------------------------------------------------
def _streams(case):
    rng = random.Random(case["layout"])
    n, top = case["streams"], case["samples"]
    lengths = [rng.randint((top + 1) // 2, top) if case["ragged"] else top for _ in range(n)]
    windows = [case["window"] or rng.choice(CLASSES[1:] if case["kind"] == "serve" else CLASSES) for _ in range(n)]
    mixed = case["mode"] == "mixed"
    modes = [rng.choice([0, 1, 2]) if mixed else MODES[case["mode"]] for _ in range(n)]
    ks = [float(np.float32(rng.uniform(2.5, 5.0))) if mixed else 3.0 for _ in range(n)]
    return lengths, windows, ks, modes


def _outputs(modes):
    """Threshold multiples and modes of the three outputs of a "multi" case."""
    other = {0: 1, 1: 0, 2: 0}
    return [3.0, 5.0, 3.0], [modes[0], modes[0], other[modes[0]]]


def _inputs(case, seed, lengths):
    """Packed streams on the GPU: Gaussian noise with impulsive bursts, the
    distributions of the benchmark's workloads."""
    rng = random.Random(case["layout"] + 1)
    specs = []
    for length in lengths:
        if case["dtype"] == "i16":
            specs.append(synth.StreamSpec(length, 8192, 3.0, 0, 400.0, 0.01, 32, 32, "i16"))
        else:
            specs.append(synth.StreamSpec(length, 4096, 3.0, 0, rng.uniform(6.0, 20.0), rng.uniform(0.001, 0.02), 8, 512))
    return synth.gen_packed(specs, seed=seed % (1 << 31), tag=77, device=torch.device("cuda", 0))


def prepare(case, seed):
    lengths, windows, ks, modes = _streams(case)
    kind = case["kind"]
    x = _inputs(case, seed, lengths)
    s = {"kind": kind, "x": x, "lengths": np.array(lengths, np.int64), "windows": np.array(windows, np.int32),
         "k": np.array(ks, np.float32), "mode": np.array(modes, np.int32)}
    if kind in ("filter", "mom", "carry"):
        s["y"] = torch.zeros_like(x)  # padding between streams is never written
    if kind in ("mom", "carry"):
        s["mom_k"] = case["mom_k"]
    if kind == "carry":
        n, pre, dev = len(lengths), case["mom_k"] - 1, x.device
        # the streams have been running for about half a history
        g = torch.Generator(device=dev).manual_seed(seed % (1 << 31) + 1)
        s["history"] = torch.randint(4, 16, (n, pre), generator=g, device=dev, dtype=torch.uint8)
        s["history_len"] = torch.full((n,), pre // 2, dtype=torch.int32, device=dev)
        s["abs_base"] = torch.tensor([w * (pre // 2) for w in windows], dtype=torch.int64, device=dev)
    if kind == "multi":
        s["ks"], s["modes"] = _outputs(modes)
        s["ys"] = [torch.zeros_like(x) for _ in range(3)]
    if kind == "power":
        # the filtered batch: bursts clipped away, as a filter leaves it
        top = 24 if case["dtype"] == "i8" else 1200
        s["filtered"] = x.clamp(-top, top)
        s["block"] = case["block"]
    if kind == "serve":
        offs, _ = synth.packed_offsets(lengths)
        srv = rfi.Server(elem_size=1, max_streams=len(lengths), max_inflight=256, max_batch=64, seed=NOISE_SEED, n_lanes=2)
        for i, (w, k, m) in enumerate(zip(windows, ks, modes)):
            srv.add_stream(i, w, k, m)
        room = [(srv.out_elems(i, n) + 63) // 64 * 64 for i, n in enumerate(lengths)]
        recs = [srv.stats_entries(i, n) for i, n in enumerate(lengths)]
        s["server"] = srv
        s["out"] = torch.zeros(sum(room), dtype=torch.int8, device=x.device)
        s["stats"] = torch.zeros((sum(recs), 4), dtype=torch.int32, device=x.device)
        s["ids"] = np.arange(len(lengths), dtype=np.uint32)
        s["arrival"] = np.zeros(len(lengths), np.int64)
        s["in_ptr"] = np.array([x.data_ptr() + o for o in offs], np.uint64)
        s["out_ptr"] = np.array([s["out"].data_ptr() + sum(room[:i]) for i in range(len(room))], np.uint64)
        s["stats_ptr"] = np.array([s["stats"].data_ptr() + 16 * sum(recs[:i]) for i in range(len(recs))], np.uint64)
    return s


def run(s):
    kind = s["kind"]
    if kind == "filter":
        y, st = _lib.mad_filter(s["x"], s["lengths"], s["windows"], s["k"], s["mode"], seed=NOISE_SEED, y=s["y"])
        return {"y": y, "stats": st}
    if kind == "multi":
        ys, sts = _lib.mad_filter_multi(s["x"], s["lengths"], s["windows"], s["ks"], s["modes"], seed=NOISE_SEED, ys=s["ys"])
        return {"y": ys, "stats": sts}
    if kind == "mom":
        y, st = _lib.mom_filter(s["x"], s["lengths"], s["windows"], s["k"], s["mode"], s["mom_k"], seed=NOISE_SEED, y=s["y"])
        return {"y": y, "stats": st}
    if kind == "carry":
        y, st = _lib.mom_filter_carry(s["x"], s["lengths"], s["windows"], s["k"], s["mode"], s["mom_k"], s["abs_base"],
                                      s["history"], s["history_len"], seed=NOISE_SEED, y=s["y"])
        return {"y": y, "stats": st, "history": s["history"], "history_len": s["history_len"]}
    if kind == "power":
        pu = _lib.block_power(s["x"], s["lengths"], s["block"])
        pf = _lib.block_power(s["filtered"], s["lengths"], s["block"])
        return {"power": pu, "filtered": pf, "improvement": _lib.improvement(pu, pf, s["lengths"], s["block"], SEGMENT)}
    _, emitted = s["server"].replay_ptrs(s["ids"], s["arrival"], s["in_ptr"], s["out_ptr"], s["lengths"], s["stats_ptr"])
    return {"y": s["out"], "stats": s["stats"], "emitted": emitted}


def work(case):
    lengths, windows, _, _ = _streams(case)
    elem = 2 if case["dtype"] == "i16" else 1
    samples = sum(lengths)
    records = 16 * sum(-(-n // w) for n, w in zip(lengths, windows))
    kind = case["kind"]
    if kind == "power":
        moved = 2 * samples * elem + 2 * 8 * sum(-(-n // case["block"]) for n in lengths) + 24 * len(lengths)
    elif kind == "multi":
        moved = 4 * samples + 3 * records
    elif kind == "carry":
        moved = 2 * samples + records + 2 * len(lengths) * (case["mom_k"] - 1)
    else:
        moved = 2 * samples * elem + records
    return {"bytes": moved, "flops": 0}


# ---------------------------------------------------------------------------
# The results in 64 bits, from the definitions alone.
# ---------------------------------------------------------------------------
def _windows_of(v, w):
    """The stream's windows as rows: the whole ones, then the short last one."""
    whole = v.numel() // w * w
    parts = [v[:whole].view(-1, w)] if whole else []
    return parts + ([v[whole:].view(1, -1)] if whole < v.numel() else [])


def _lower_median(rows):
    return torch.kthvalue(rows, (rows.shape[1] - 1) // 2 + 1, dim=1).values


def _bits(t):
    return t.view(torch.int32)


def _median_mad(v, w):
    med, mad = [], []
    for rows in _windows_of(v, w):
        m = _lower_median(rows)
        med.append(m)
        mad.append(_lower_median((rows - m[:, None]).abs()))
    return torch.cat(med), torch.cat(mad)


def _replace(v, w, med, scale, mad, k, mode, limits):
    """The filtered stream (None where noise is drawn) and its statistics."""
    t = torch.full_like(scale, k, dtype=torch.float32) * (torch.full_like(scale, 1.4826, dtype=torch.float32) * scale.float())
    edge = t.double().floor().long()
    out, flagged, at = [], [], 0
    for rows in _windows_of(v, w):
        m, e = med[at:at + len(rows), None], edge[at:at + len(rows), None]
        at += len(rows)
        hit = (rows - m).abs() > e
        flagged.append(hit.sum(1))
        if mode == 0:
            out.append(rows.masked_fill(hit, 0).reshape(-1))
        elif mode == 1:
            out.append(torch.maximum(torch.minimum(rows, m + e), m - e).clamp(*limits).reshape(-1))
    st = torch.stack([med.int(), mad.int(), torch.cat(flagged).int(), _bits(t)], 1)
    return (torch.cat(out) if out else None), st


def _rolling(mads, k):
    """Lower median of the last k entries up to each one (MADs below 256)."""
    hot = torch.zeros((len(mads) + 1, 256), dtype=torch.int64, device=mads.device)
    hot[1:].scatter_(1, mads[:, None], 1)
    below = hot.cumsum(0).cumsum(1)
    b = torch.arange(1, len(mads) + 1, device=mads.device)
    a = (b - k).clamp_min(0)
    return ((below[b] - below[a]) < ((b - a - 1) // 2 + 1)[:, None]).sum(1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "serve":  # what a pass emits depends on the blocks before it
        return None
    lengths, windows, ks, modes = _streams(case)
    s = prepare(case, seed)
    offs, _ = synth.packed_offsets(lengths)
    if kind == "power":
        def power(x):
            return torch.cat([torch.stack([b.long().square().sum() for b in x[o:o + n].split(case["block"])])
                              for o, n in zip(offs, lengths)])
        pu, pf = power(s["x"]), power(s["filtered"])
        rows, at = [], 0
        for n in lengths:
            whole, count = n // case["block"], -(-n // case["block"])
            r = []
            for p in (pu, pf):
                seg = p[at:at + whole // SEGMENT * SEGMENT].double().view(-1, SEGMENT)
                r.append((seg.std(1, unbiased=False) / seg.mean(1)).mean())
            rows.append(torch.stack(r + [10 * torch.log10(r[0] / r[1])]))
            at += count
        return {"power": pu, "filtered": pf, "improvement": torch.stack(rows)}
    limits = (-32768, 32767) if case["dtype"] == "i16" else (-128, 127)
    n_out = 3 if kind == "multi" else 1
    ys = [torch.zeros_like(s["x"]) for _ in range(n_out)]
    sts = [[] for _ in range(n_out)]
    drawn = [False] * n_out
    for i, (o, n, w) in enumerate(zip(offs, lengths, windows)):
        v = s["x"][o:o + n].long()
        med, mad = _median_mad(v, w)
        scale = mad
        if kind in ("mom", "carry"):
            past = s["history"][i, (case["mom_k"] - 1) - (case["mom_k"] - 1) // 2:].long() if kind == "carry" else mad[:0]
            scale = _rolling(torch.cat([past, mad]), case["mom_k"])[len(past):]
        for j in range(n_out):
            k, m = (_outputs(modes)[0][j], _outputs(modes)[1][j]) if kind == "multi" else (ks[i], modes[i])
            y, st = _replace(v, w, med, scale, mad, k, m, limits)
            sts[j].append(st)
            if y is None:
                drawn[j] = True
            else:
                ys[j][o:o + n] = y.to(ys[j].dtype)
    ys = [None if d else y for y, d in zip(ys, drawn)]
    sts = [torch.cat(t) for t in sts]
    if kind == "multi":
        return {"y": ys, "stats": sts}
    out = {"y": ys[0], "stats": sts[0]}
    if kind == "carry":
        out.update(history=None, history_len=None)
    return out
