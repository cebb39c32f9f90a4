"""The native operator binding refuses what it cannot pass on, with a Python error and before any launch (no GPU needed)."""
import os
import subprocess
import sys

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


# Entry points that stand in for the library's: they return what they were given.
STAND_IN = r"""
#include <stddef.h>
extern "C" {
int conv(const void*, int, const float*, const float*, const float*, const float*, int groups, int silu, const void*, const float*, const void*, void*, int, int, int, int,
         int cin, int, void*) { return 10000 * cin + 100 * groups + silu; }
int adaln(const void*, int, const void*, int, const float*, float*, int, int, int, int silu, void*) { return silu; }
}
"""
CALLER = r"""
import ctypes, sys, numpy, torch
from paper_2602_00608_amd import _binding as b
class Device(torch.Tensor):   # on the device by its own account, without an address
    __torch_function__ = torch._C._disabled_torch_function_impl
    __new__ = staticmethod(lambda cls, *shape: torch.Tensor._make_wrapper_subclass(cls, shape, dtype=torch.float32, device="cuda"))
    @classmethod
    def __torch_dispatch__(cls, func, types, args=(), kwargs=None): raise RuntimeError(func)
l = ctypes.CDLL(sys.argv[1])
at = lambda name: ctypes.cast(getattr(l, name), ctypes.c_void_p).value
b.bind(0, at("conv"), at("conv"), 0, 0, 0, 0, at("adaln"))
def conv(groups, silu, x=Device(1, 2, 2, 3)): return b.conv(3, x, None, None, None, None, groups, silu, None, None, None, Device(1, 2, 2, 4), 0)
def adaln(silu): return b.adaln(Device(1, 8), Device(16, 8), None, Device(1, 16), silu, 0)
def refused(error, f, *args):
    try: f(*args)
    except error: return
    raise AssertionError((error, args))
"""


def _with_stand_in(tmp_path, body, source=STAND_IN):
    src, lib = tmp_path / "stand_in.cpp", str(tmp_path / "stand_in.so")
    src.write_text(source)
    subprocess.run(["g++", "-shared", "-fPIC", "-o", lib, str(src)], check=True)
    wmdec.lib()   # (built)
    r = subprocess.run([sys.executable, "-c", CALLER + body, lib], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]


def test_arguments_are_converted_as_int_and_ctypes_do(tmp_path):
    _with_stand_in(tmp_path, r"""
assert conv(2, True) == 30201 and conv(numpy.int64(5), numpy.bool_(False)) == 30500 and conv(torch.tensor(4), 1) == 30401
assert conv(2 ** 32 + 7, 2) == 30702 and conv(2 ** 70 + 6, "3") == 30603 and conv(1, 0.5) == 30100 == conv(True, False)
assert conv(2, 0, Device(1, 2, 2, 3, 1)) == 30200           # channels are dimension 3
assert adaln(True) == 1 and adaln(0.5) == 0 and adaln(numpy.float32(2)) == 2
for f in (adaln, lambda silu: conv(2, silu)):
    refused(TypeError, f, None)
    refused(ValueError, f, "yes")
    refused(ValueError, f, float("nan"))
for groups in (None, 2.0, "2"): refused(TypeError, conv, groups, 1)
refused(ValueError, conv, 2, 1, Device(2, 2, 3))
""")


def test_an_exception_from_an_entry_point_becomes_a_python_error(tmp_path):
    _with_stand_in(tmp_path, r"""
import threading
def call():
    for _ in range(200): refused(RuntimeError, adaln, True)
others = [threading.Thread(target=call) for _ in range(4)]
for t in others: t.start()
call()
for t in others: t.join()
try: adaln(True)
except RuntimeError as e: assert str(e) == "no memory for it", e
""", """
#include <stdexcept>
extern "C" {
int conv() { return 0; }
int adaln() { throw std::runtime_error("no memory for it"); }
}
""")
