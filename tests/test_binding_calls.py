"""How the binding hands the arguments of a call over (csrc/pycall.cpp), seen from a C callback in the library's place."""
import ctypes
import os
import re
import subprocess
import sys
import sysconfig

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


def test_threads_that_make_the_first_call_together(monkeypatch):
    """Between any two bytecodes of the first call that asks for the stream, another thread's call finds getters it can use."""
    for name, value in (("_cuda_getCurrentRawStream", lambda device: 70 + device), ("_cuda_getDevice", lambda: 7)):
        monkeypatch.setattr(torch._C, name, value, raising=False)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(B, "_raw_stream", None)
    monkeypatch.setattr(B, "_device", None)
    seen = 0

    def first_call(interrupted_at):
        nonlocal seen
        B._raw_stream = B._device = None
        seen = 0

        def trace(frame, event, arg):
            nonlocal seen
            if frame.f_code is not B._current_stream.__code__:
                return None
            frame.f_trace_opcodes = True
            if event == "opcode":
                seen += 1
                if seen == interrupted_at:
                    assert B._current_stream() == 77              # (not traced in here)
            return trace

        before = sys.gettrace()
        sys.settrace(trace)
        try:
            assert B._current_stream() == 77
        finally:
            sys.settrace(before)

    first_call(0)
    assert seen > 20
    for at in range(1, seen + 1):
        first_call(at)


def test_a_stream_without_a_handle_is_the_default_one():
    assert B._on(type("S", (), {"cuda_stream": None})()) == 0


ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_caller_is_for_one_python(call):
    """Its name says which: an extension of another interpreter's ABI must not be loaded."""
    from paper_2407_00079_amd import _mccall, build
    assert _mccall.__file__ == build.CALLER and build.CALLER.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    assert not os.path.exists(os.path.join(build.PKG, "_mccall.so"))


def test_without_a_caller_calls_go_through_ctypes():
    """As from an interpreter it was not built for: every argument check of the library is reached with the same results.  (No
    call here passes all of them with anything to do: nothing is launched, with or without a GPU.)"""
    code = """
import sys
sys.path.insert(0, %r)
sys.modules["paper_2407_00079_amd._mccall"] = None if len(sys.argv) > 1 else __import__("paper_2407_00079_amd._mccall")._mccall
from paper_2407_00079_amd import binding as B
class S: cuda_stream = 0
class T:
    nbytes = 8
    def data_ptr(self): return 1 << 40
    def dim(self): return 2
    def size(self, i): return 4
p, t, s, plan = B.attn_params(8, 2, 128, 16, 64, "bf16"), T(), S(), B.McAttnPlan()
def status(f):
    try:
        return f()
    except B.McError as e:
        return str(e)
    except Exception as e:
        return "refused"
lens = [[16, 3], [5, 2]]
for f in (lambda: B.mc_prefill_attn_paged(p, t, t, t, t, *lens, t, None, t, s), lambda: B.mc_prefill_attn_paged(p, t, t, t, t, [16, 300], [5, 2], t, None, t, s),
          lambda: B.mc_prefill_attn_paged(None, t, t, t, t, *lens, t, None, t, s), lambda: B.mc_prefill_attn_auto(p, t, t, t, t, (16, 3), [5, 2], t, t, None, s),
          lambda: B.mc_prefill_attn_paged(p, t, t, t, t, [0], [0], t, None, t, s), lambda: B.mc_prefill_attn_paged_noalloc(p, t, t, t, t, [-1], [5], t, None, s),
          lambda: B.mc_prefill_attn_run(p, plan, t, t, t, t, t, None, t, s), lambda: B.mc_kv_append_run(p, plan, t, t, t, t, t, t, s),
          lambda: B.mc_kv_append_paged(p, t, t, t, t, t, *lens, t, s), lambda: B.mc_kv_append_paged(p, t, None, t, t, t, *lens, t, s),
          lambda: B.mc_kv_pack_layer(t, t, 4, 33, t, 2, t, t, s), lambda: B.mc_kv_pack_layer(t, t, 4, 32.0, t, 2, t, t, s),
          lambda: B.mc_kv_unpack_layer(t, t, 4, 32, None, 2, t, t, s), lambda: B.mc_kv_page_order(t, -1, t, s),
          lambda: B.mc_kv_pack_layer_ordered(t, t, -4, 32, t, t, 2, t, t, s), lambda: B.mc_kv_unpack_layer_ordered(t, t, 4, 24, t, None, 2, t, t, s),
          lambda: B.mc_prefix_hash(t, [0, 700], 512, t, t, s), lambda: B.mc_prefix_hash(t, [0, -7], 512, t, t, s), lambda: B.mc_prefix_hash(t, [0, "x"], 512, t, t, s),
          lambda: B.mc_prefix_match(t, [0, 2], t, [0, -9], t, t, t, t, s), lambda: B.mc_prefix_match(t, [0, 2], None, [0, 9], t, t, t, t, s)):
    print(status(f))
print(B._call.__name__, file=sys.stderr)
""" % ROOT
    native, by_ctypes = (subprocess.run([sys.executable, "-c", code, *arg], capture_output=True, text=True, timeout=120) for arg in ([], ["x"]))
    assert native.returncode == 0 and by_ctypes.returncode == 0, (native.stderr, by_ctypes.stderr)
    assert native.stderr.split()[-1] == "call" and by_ctypes.stderr.split()[-1] == "_call_by_ctypes"
    assert native.stdout == by_ctypes.stdout and len(native.stdout.splitlines()) == 21, (native.stdout, by_ctypes.stdout)
    assert "mc_status 7" not in native.stdout and len(set(native.stdout.splitlines())) > 6         # statuses of several kinds, and refusals


def declarations():
    """The parameters that include/mc.h declares: function -> (type, name) of each."""
    text = re.sub(r"/\*.*?\*/", "", open(os.path.join(ROOT, "include", "mc.h")).read(), flags=re.S)
    found = re.findall(r"\b(mc_[a-z_0-9]+)\s*\(([^)]*)\)\s*;", text)
    return {f: [re.fullmatch(r"(.*?)\s*(\w+)", p.strip(), flags=re.S).groups() for p in params.split(",")] for f, params in found}


def test_the_kinds_are_those_of_the_declared_parameters():
    """One letter a parameter: a call with fewer would leave the rest of them zero, with no one to notice."""
    host = {"prefix_lens", "new_lens", "tok_offsets", "key_offsets", "cache_offsets"}
    declared = declarations()
    assert len(B._KINDS) == 13
    for function, kinds in B._KINDS.items():
        want = ""
        for type_, name in declared[function]:
            if name in host:
                want += {"const int32_t*": "I", "const int64_t*": "Q"}[type_]
            elif type_.startswith("const mc_attn_"):
                want += "s"
            else:                                             # the stream's handle comes as an integer
                want += "p" if type_.endswith("*") and name != "hip_stream" else "i"
        assert kinds == want and len(getattr(B.lib(), function).argtypes) == len(want), function
