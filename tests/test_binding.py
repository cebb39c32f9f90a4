"""The native operator binding refuses what it cannot pass on, with a Python error and before any launch (no GPU needed)."""
import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode

from paper_2602_00608_amd import wmdec


def _stats(x, groups=2, stream=0):
    f = torch.zeros(2)
    return wmdec._ops().gn_stats(x, groups, 1e-6, f, f, f, stream)


def _fake(*shape, dtype=torch.float32):
    with FakeTensorMode():
        return torch.empty(shape, dtype=dtype, device="cuda")


@pytest.mark.parametrize("call, error", [
    (lambda: wmdec._ops().gn_stats(), TypeError),                      # number of arguments
    (lambda: wmdec._ops().bind(*range(7)), TypeError),
    (lambda: _stats(3), TypeError),                                    # no tensor
    (lambda: _stats(torch.zeros(1, 2, 2, 4)), AssertionError),         # not on the device
    (lambda: wmdec._ops().upconv(None, None, None, None, 0), TypeError),
    (lambda: torch.vmap(_stats)(_fake(3, 1, 2, 2, 4)), RuntimeError),  # a tensor without an address: torch throws
    (lambda: _stats(_fake(1, 4, 2, 2).permute(0, 2, 3, 1)), AssertionError),   # not contiguous
], ids=["count", "bind", "no-tensor", "host", "none", "no-storage", "strided"])
def test_refused_with_an_error(call, error):
    with pytest.raises(error):
        call()
