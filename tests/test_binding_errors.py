"""What the Python binding passes on for the library to refuse, and errors
that are not the library's (host only where no device is named)."""
import pytest
import torch

import paper_1710_08576_amd as rfi
from paper_1710_08576_amd import synth


class _NullStream:
    cuda_stream = 0


@pytest.mark.parametrize("missing", ["power_u", "power_f"])
def test_improvement_without_powers(missing):
    args = {"power_u": torch.ones(8, dtype=torch.int64), "power_f": torch.ones(8, dtype=torch.int64)}
    args[missing] = None
    with pytest.raises(rfi.RfiError) as e:
        rfi.improvement(*args.values(), [8], 1, 4, out=torch.empty((1, 3), dtype=torch.float64), stream=_NullStream())
    assert e.value.status == -1


@pytest.mark.gpu
def test_errors_left_by_the_program(gpu):
    """A HIP error that the program left (and did not ask for) is not the
    launches': every entry point answers as without it."""
    L = [40_000, 40_000]
    x8 = synth.gen_packed([synth.StreamSpec(n, 4096, 3.0, 2, 9.0, 0.02, 8, 600) for n in L], 1, 31).to(gpu)
    x16 = synth.gen_packed([synth.StreamSpec(n, 8192, 3.0, 2, 400.0, 0.02, 8, 600, "i16") for n in L], 1, 31).to(gpu)
    y8, y16, hip = torch.zeros_like(x8), torch.zeros_like(x16), rfi.load()
    power = torch.ones(80, dtype=torch.int64, device=gpu)
    room = torch.empty(128, dtype=torch.float64, device=gpu)
    calls = [lambda x=x, y=y, W=W, m=m: rfi.mad_filter(x, L, [W] * 2, [3.0] * 2, [m] * 2, y=y)
             for x, y in ((x8, y8), (x16, y16)) for W in (100, 4096, 8192, 9000, 20_000, 40_000) for m in (1, 2)]
    calls += [lambda: rfi.mom_filter(x8, L, [700] * 2, [3.0] * 2, [2] * 2, 5, y=y8),
              lambda: rfi.mad_filter_multi(x8, L, [700] * 2, [3.0, 2.0], [0, 1]),
              lambda: rfi.mad_filter_noalloc(x8, L, [700] * 2, [3.0] * 2, [2] * 2, y=y8),
              lambda: rfi.block_power(x8, L, 1000), lambda: rfi.block_power(x16, L, 40_000),
              lambda: rfi.improvement(power, power, L, 1000, 4, out=room[:6].view(2, 3))]
    srv = rfi.Server(elem_size=1, max_streams=2, n_lanes=1)
    srv.add_stream(0, 4096, 3.0, 2)

    def serve():
        t = srv.submit(0, x8[:40_000], y8)
        srv.dispatch()
        srv.sync()
        assert srv.poll(t)[0]

    for call in calls + [serve]:
        call()  # work tables, lanes and torch's pools are there
        torch.cuda.synchronize()
        assert hip.hipSetDevice(9999) != 0
        try:
            call()
        finally:
            hip.hipGetLastError()
        torch.cuda.synchronize()
    srv.close()
