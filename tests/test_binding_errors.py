"""What the Python binding passes on for the library to refuse, and errors
that are not the library's (host only where no device is named)."""
import pytest
import torch

import paper_1710_08576_amd as rfi


class _NullStream:
    cuda_stream = 0


@pytest.mark.parametrize("missing", ["power_u", "power_f"])
def test_improvement_without_powers(missing):
    args = {"power_u": torch.ones(8, dtype=torch.int64), "power_f": torch.ones(8, dtype=torch.int64)}
    args[missing] = None
    with pytest.raises(rfi.RfiError) as e:
        rfi.improvement(*args.values(), [8], 1, 4, out=torch.empty((1, 3), dtype=torch.float64), stream=_NullStream())
    assert e.value.status == -1
