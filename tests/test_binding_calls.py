"""How the binding hands the arguments of a call over (csrc/pycall.cpp), seen from a C callback in the library's place."""
import ctypes
import os

import numpy as np
import pytest
import torch

from paper_2407_00079_amd import binding as B


@pytest.fixture(scope="module")
def call():
    B.lib()
    from paper_2407_00079_amd import _mccall
    return _mccall.call


def spy(n, look=lambda a: a):
    """A C function of n 64-bit integers and a list that receives what it was called with."""
    seen = []

    def f(*a):
        seen.append(look(a))
        return len(seen) - 1

    c = ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_int64] * n)(f)
    return c, ctypes.cast(c, ctypes.c_void_p).value, seen


class Tensor:
    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        return self.at


def test_every_kind_arrives(call):
    params = B.attn_params(8, 2, 128, 16, 64, "bf16")

    def look(a):
        i32, i64 = (ctypes.c_int32 * 3).from_address(a[5]), (ctypes.c_int64 * 2).from_address(a[6])
        return a[:5], list(i32), list(i64), a[7:]

    keep, at, seen = spy(14, look)
    odd = [np.int64(2 ** 40), 7.9]                            # as int() takes them
    args = (params, Tensor(2 ** 47 + 16), None, -1, np.int32(5), [3, -4, 2 ** 32 + 6], odd, B._Ints("i", (1, 2), 2), 1, 2, 3, 4, 5, 6)
    assert call(at, "sppiiIQIiiiiii", *args) == 0 and call(at, "sppiiIQIiiiiii", *args) == 1
    first, i32, i64, rest = seen[0]
    assert first == (ctypes.addressof(params), 2 ** 47 + 16, 0, -1, 5)
    assert i32 == [3, -4, 6] and i64 == [2 ** 40, 7]
    assert rest == (args[7].at, 1, 2, 3, 4, 5, 6)


@pytest.mark.parametrize("kinds,args,error", [
    ("p", (5,), AttributeError), ("p", ([1],), AttributeError),        # an address is no tensor
    ("i", (1.0,), TypeError), ("i", ("1",), TypeError), ("i", (None,), TypeError), ("i", ([1],), TypeError),
    ("s", (7,), TypeError),
    ("I", ((1, 2),), TypeError), ("I", (["x"],), ValueError), ("Q", ([None],), TypeError),
    ("IQI", ([1], [2], [3]), TypeError),
    ("i", (1, 2), TypeError), ("ii", (1,), TypeError), ("i" * 21, (0,) * 21, TypeError),
])
def test_what_does_not_fit_is_refused_before_the_call(call, kinds, args, error):
    keep, at, seen = spy(1)
    with pytest.raises(error):
        call(at, kinds, *args)
    assert not seen
    with pytest.raises(TypeError):
        call(0, "i", 1)


def test_lists_and_what_stands_for_them():
    same = [4, 5]
    assert B._ints("i", same, 2) is same
    for values, n in (((4, 5), 2), (np.array([4, 5]), 2), ([4], 3), ([], 0), (range(2), 2)):
        assert isinstance(B._ints("i", values, n), B._Ints)
    with pytest.raises(IndexError):
        B._ints("i", [1, 2, 3], 2)
    with pytest.raises(TypeError):
        B.mc_prefill_attn_run(B.attn_params(8, 1, 128, 16, 4, "bf16"), None, None, None, None, None, None, None, None, 0)
    with pytest.raises(B.McError):
        B.mc_kv_pack_layer(None, None, 4, 32, None, 1, None, None, type("S", (), {"cuda_stream": 0})())


def test_a_forked_child_asks_torch_for_its_stream(monkeypatch):
    """The parent's stream getters are not used in a child: torch refuses the GPU there once the parent has used it."""
    for name, value in (("_cuda_getCurrentRawStream", lambda device: 70 + device), ("_cuda_getDevice", lambda: 7)):
        monkeypatch.setattr(torch._C, name, value, raising=False)
    monkeypatch.setattr(B, "_raw_stream", None)
    monkeypatch.setattr(B, "_device", None)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    assert B._on(None) == 77 and B._on(None) == 77

    def refused():
        raise RuntimeError("no GPU in a forked child")

    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: False)
    monkeypatch.setattr(torch.cuda, "current_stream", refused)
    pid = os.fork()
    if pid == 0:
        status = 1
        try:
            B._on(None)
        except RuntimeError:
            status = 0
        finally:
            os._exit(status)
    assert os.waitpid(pid, 0)[1] == 0
    assert B._on(None) == 77                                  # the parent's stay


def test_a_stream_without_a_handle_is_the_default_one():
    assert B._on(type("S", (), {"cuda_stream": None})()) == 0
