"""The native half of the binding (csrc/va_host.cpp), built for CPU tensors (marshalling_check.cpp) and bound to functions that
only note what they are called with: what it allocates and how, what it refuses, and which errors come out of it."""
import ctypes
import importlib.machinery
import importlib.util
import os
import types

import pytest
import torch
from torch.utils._python_dispatch import TorchDispatchMode

from paper_2605_08962_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
T, HQ, HKV, D, WORKSPACE = 70, 2, 1, 64, 4096


@pytest.fixture(scope="module")
def module(tmp_path_factory):
    path = build.compile_host(os.path.join(HERE, "marshalling_check.cpp"),
                              str(tmp_path_factory.mktemp("host") / "marshalling_check.so"))
    loader = importlib.machinery.ExtensionFileLoader("marshalling_check", path)
    m = importlib.util.module_from_spec(importlib.util.spec_from_loader("marshalling_check", loader))
    loader.exec_module(m)
    return m


@pytest.fixture
def host(module):
    """The module, bound to functions that succeed; `calls` holds the arguments of each."""
    calls, vp, sz = [], ctypes.c_void_p, ctypes.c_size_t
    size = ctypes.CFUNCTYPE(sz, vp)(lambda p: WORKSPACE)

    def noted(name):
        def f(*args):
            calls.append((name, args))
            return 0
        return f
    fwd = ctypes.CFUNCTYPE(ctypes.c_int, *[vp] * 8, sz, vp)(noted("fwd"))
    bwd = ctypes.CFUNCTYPE(ctypes.c_int, *[vp] * 12, sz, vp)(noted("bwd"))
    merge = ctypes.CFUNCTYPE(ctypes.c_int, vp, ctypes.c_int32, *[vp] * 5)(noted("merge"))
    functions = (size, size, fwd, bwd, merge)
    module.bind(*(ctypes.cast(f, vp).value for f in functions))
    module.set_current_stream(0)
    module.watch(False)
    yield types.SimpleNamespace(fwd=module.fwd, bwd=module.bwd, merge=module.merge, watch=module.watch,
                                set_current_stream=module.set_current_stream, calls=calls, keep=functions)
    module.watch(False)


def _attn(**other):
    """Arguments of a forward and of a backward on one good batch, some of them replaced."""
    bf = lambda h: torch.zeros((T, h, D), dtype=torch.bfloat16)  # noqa: E731
    a = dict(dout=bf(HQ), q=bf(HQ), k=bf(HKV), v=bf(HKV), o=bf(HQ), lse=torch.zeros(HQ, T), cu=torch.tensor([0, 30, T]).int(),
             out=None, out_lse=None, dq=None, dk=None, dv=None, workspace=None, stream=None)
    assert not other.keys() - a.keys()
    a.update(other)
    return a


# Each returns the call, its arguments made.
def _fwd(host, **other):
    a = _attn(**other)
    return lambda: host.fwd(a["q"], a["k"], a["v"], a["cu"], True, 0.1, a["out"], a["out_lse"], a["workspace"], a["stream"], 0, 0)


def _bwd(host, **other):
    a = _attn(**other)
    return lambda: host.bwd(a["dout"], a["q"], a["k"], a["v"], a["o"], a["lse"], a["cu"], True, 0.1, a["dq"], a["dk"], a["dv"],
                            a["workspace"], a["stream"], 0, 0)


def _merge(host, out=None, out_lse=None, stream=None):
    parts, lse = torch.zeros((2, T, HQ, D), dtype=torch.bfloat16), torch.zeros(2, HQ, T)
    return lambda: host.merge(parts, lse, out, out_lse, stream)


CALLS = pytest.mark.parametrize("make", [_fwd, _bwd, _merge])


@CALLS
def test_a_good_call_goes_through(host, make):
    done = make(host)()
    assert type(done) is tuple and [name for name, _ in host.calls] == [make.__name__[1:]]
    assert done[0].shape == (T, HQ, D) and done[0].dtype == torch.bfloat16


@CALLS
def test_out_of_memory_is_what_torch_makes_of_it(host, make):
    call = make(host)
    host.watch(True)
    with pytest.raises(torch.OutOfMemoryError, match="the test has no memory"):
        call()
    assert not host.calls


@CALLS
def test_a_python_error_inside_an_allocation_stays_what_it_is(host, make):
    class Refuses(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            raise KeyError("no allocations here")

    call = make(host)
    with Refuses(), pytest.raises(KeyError, match="no allocations here"):
        call()


@CALLS
def test_allocations_leave_the_interpreter_to_other_threads(host, make):
    """As torch.empty does: one that has to go to the driver may take milliseconds."""
    call = make(host)
    host.watch(False)
    call()
    with_lock, without_lock = host.watch(False)
    assert with_lock == 0 and without_lock >= 2
