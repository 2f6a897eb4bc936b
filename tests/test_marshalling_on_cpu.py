"""The native half of the binding (csrc/va_host.cpp), built for CPU tensors (marshalling_check.cpp) and bound to functions that
only note what they are called with: what it allocates and how, what it refuses, and which errors come out of it.  The same
refusals of the Python half, by name, with a library that notes its calls."""
import contextlib
import ctypes
import importlib.machinery
import importlib.util
import os
import types
import warnings

import pytest
import torch
from torch.utils._python_dispatch import TorchDispatchMode

from paper_2605_08962_amd import binding, build

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


def _bf(*shape):
    return torch.zeros(shape, dtype=torch.bfloat16)


# What a call may not be given: (call, replaced arguments, the name that the Python half refuses it by).
BAD = [
    # k and v of another length or head_dim than q: read past their ends
    (_bwd, dict(k=_bf(T - 1, HKV, D), v=_bf(T - 1, HKV, D)), "k and v"),
    (_bwd, dict(k=_bf(T, HKV, 32), v=_bf(T, HKV, 32)), "k and v"),
    (_bwd, dict(k=_bf(T, HKV), v=_bf(T, HKV)), "k and v"),
    (_bwd, dict(lse=torch.zeros(HQ, T - 1)), "lse"),
    (_bwd, dict(lse=torch.zeros(T)), "lse"),
    # results: too small, of another type, with gaps
    (_fwd, dict(out=_bf(T - 1, HQ, D)), "out"),
    (_fwd, dict(out=torch.zeros(T, HQ, D)), "out"),
    (_fwd, dict(out=_bf(T, HQ, 2 * D)[:, :, :D]), "out"),
    (_fwd, dict(out_lse=torch.zeros(HQ, T - 1)), "lse"),
    (_fwd, dict(out_lse=torch.zeros(HQ, T, dtype=torch.float64)), "lse"),
    (_bwd, dict(dq=_bf(T, HQ, D - 8)), "dq"),
    (_bwd, dict(dk=_bf(T, HQ, D).float()), "dk"),
    (_bwd, dict(dv=_bf(HKV, T, D)[:, ::2]), "dv"),
    (_merge, dict(out=_bf(T, 1, D)), "out"),
    (_merge, dict(out_lse=torch.zeros(1, T)), "lse"),
    # a workspace whose elements do not lie side by side
    (_fwd, dict(workspace=torch.zeros(1, dtype=torch.uint8).expand(1 << 20)), "workspace"),
    (_bwd, dict(workspace=torch.zeros(2 * WORKSPACE, dtype=torch.uint8)[::2]), "workspace"),
]
# And what it may: a buffer that is larger than the result, or shaped otherwise.
GOOD = [
    (_fwd, dict(out=_bf(T + 9, HQ, D), out_lse=torch.zeros(HQ * T + 3))),
    (_fwd, dict(out=_bf(T, HQ * D), workspace=torch.zeros(WORKSPACE))),
    (_bwd, dict(dq=_bf(T * HQ * D), dk=_bf(T + 1, HKV, D), lse=torch.zeros(HQ * T))),
    (_merge, dict(out=_bf(T + 9, HQ, D), out_lse=torch.zeros(HQ * T + 3))),
]


@pytest.mark.parametrize("make,other,name", BAD)
def test_the_native_half_refuses_what_would_leave_its_buffers(host, make, other, name):
    assert make(host, **other)() is NotImplemented
    assert not host.calls


@pytest.mark.parametrize("make,other", GOOD)
def test_the_native_half_takes_larger_buffers(host, make, other):
    assert type(make(host, **other)()) is tuple and len(host.calls) == 1


@pytest.fixture
def python_half(host, monkeypatch):
    """Something with the native half's call signatures that goes through the Python half."""
    never = lambda *a: NotImplemented  # noqa: E731
    monkeypatch.setattr(binding, "_host", types.SimpleNamespace(fwd=never, bwd=never, merge=never))
    calls = []
    noted = lambda name: lambda *a: calls.append(name) or 0  # noqa: E731
    size = lambda p: WORKSPACE  # noqa: E731
    lib = types.SimpleNamespace(varlen_attn_fwd=noted("fwd"), varlen_attn_bwd=noted("bwd"), varlen_attn_merge=noted("merge"),
                                varlen_attn_fwd_workspace_bytes=size, varlen_attn_bwd_workspace_bytes=size)
    monkeypatch.setattr(binding, "load", lambda: lib)
    at, made = [0], []  # the current stream's handle; (who, stream then current) of every allocation and record

    class Stream:
        def __init__(self, handle, device=None):
            self.cuda_stream = handle

    @contextlib.contextmanager
    def on(stream):
        was, at[0] = at[0], stream.cuda_stream
        yield
        at[0] = was

    class Allocations(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            if "empty" in str(func):
                made.append(("empty", at[0]))
            return func(*args, **(kwargs or {}))
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: Stream(at[0]))
    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch.cuda, "Stream", Stream)
    monkeypatch.setattr(torch.cuda, "ExternalStream", Stream)
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda t, s: made.append(("record", s.cuda_stream)))
    monkeypatch.setattr(torch.Tensor, "is_cuda", property(lambda t: True))
    kw = lambda *names: lambda a: dict(zip(names, a))  # noqa: E731
    fwd, bwd = kw("out", "lse", "workspace", "stream"), kw("dq", "dk", "dv", "workspace", "stream")
    return types.SimpleNamespace(
        fwd=lambda *a: binding.varlen_attn_fwd(*a[:6], **fwd(a[6:10])),
        bwd=lambda *a: binding.varlen_attn_bwd(*a[:9], **bwd(a[9:14])),
        merge=lambda *a: binding.varlen_attn_merge(*a[:4], stream=a[4]), calls=calls, made=made, at=at, Stream=Stream,
        allocations=Allocations)


@pytest.mark.parametrize("make,other,name", BAD)
def test_the_python_half_refuses_the_same_by_name(python_half, make, other, name):
    with pytest.raises(ValueError, match=f"^{name} must"):
        make(python_half, **other)()
    assert not python_half.calls


@pytest.mark.parametrize("make,other", GOOD)
def test_the_python_half_takes_the_same(python_half, make, other):
    assert type(make(python_half, **other)()) is tuple and len(python_half.calls) == 1


# Scratch that a call allocates for itself is given back when the call returns, while its kernels may still run: it has to come
# from the pool of the stream they run on, where what is given back is reused behind them and what is taken is free.
GIVEN = {_fwd: lambda: dict(out=_bf(T, HQ, D), out_lse=torch.zeros(HQ, T), workspace=torch.zeros(WORKSPACE)),
         _bwd: lambda: dict(dq=_bf(T, HQ, D), dk=_bf(T, HKV, D), dv=_bf(T, HKV, D), workspace=torch.zeros(WORKSPACE)),
         _merge: lambda: dict(out=_bf(T, HQ, D), out_lse=torch.zeros(HQ, T))}


@CALLS
def test_the_native_half_allocates_on_the_current_stream_only(host, make):
    host.set_current_stream(48)
    for stream, given, taken in [(None, False, True), (48, False, True), (None, True, True), (64, True, True), (64, False, False)]:
        host.calls.clear()
        done = make(host, stream=stream, **(GIVEN[make]() if given else {}))()
        assert (type(done) is tuple) == taken and (done is NotImplemented) == (not taken)
        assert [args[-1] for _, args in host.calls] == ([stream or 48] if taken else [])


@CALLS
def test_the_python_half_allocates_on_the_stream_of_the_call(python_half, make):
    python_half.at[0] = 48
    results = {_fwd: 2, _bwd: 3, _merge: 2}[make]
    for handle, given, pool in [(None, False, 48), (48, False, 48), (64, True, None), (64, False, 64)]:
        python_half.made.clear()
        call = make(python_half, stream=None if handle is None else python_half.Stream(handle), **(GIVEN[make]() if given else {}))
        with python_half.allocations():
            call()
        empties = [s for what, s in python_half.made if what == "empty"]
        assert set(empties) == (set() if given else {pool}) and (given or len(empties) >= results)
        # the results are used on the stream that was current, and may be dropped with such uses under way
        assert [s for what, s in python_half.made if what == "record"] == ([48] * results if pool == 64 else [])


def test_the_native_half_is_named_after_what_it_was_built_for(monkeypatch, tmp_path):
    """One built for another torch or interpreter, or from other sources, is another file: it is not loaded."""
    here = build.host_path()
    assert os.path.dirname(here) == build.HERE and here == build.host_path()
    names = {here}
    with monkeypatch.context() as m:
        m.setattr(torch, "__version__", "2.11.0")
        names.add(build.host_path())
    with monkeypatch.context() as m:
        m.setattr(build.sysconfig, "get_config_var", lambda name: "cpython-399")
        names.add(build.host_path())
    for name in ("va_host.cpp", "varlen_attn.h"):
        for i, path in enumerate(build.HOST_SOURCES):
            if os.path.basename(path) == name:
                changed = tmp_path / name
                changed.write_bytes(open(path, "rb").read() + b"\n")
                with monkeypatch.context() as m:
                    m.setattr(build, "HOST_SOURCES", [str(changed) if j == i else x for j, x in enumerate(build.HOST_SOURCES)])
                    names.add(build.host_path())
    assert len(names) == 5


@pytest.mark.parametrize("how", ["cannot be built", "cannot be loaded"])
def test_without_the_native_half_calls_go_through_the_python_half(monkeypatch, tmp_path, how):
    path = tmp_path / "host.so"

    def no_compiler():
        raise FileNotFoundError("g++")
    if how == "cannot be loaded":
        path.write_bytes(b"")
    monkeypatch.setattr(binding, "_host", None)
    monkeypatch.setattr(build, "host_path", lambda: str(path))
    monkeypatch.setattr(build, "build_host", no_compiler)
    q = _bf(T, HQ, D)
    with pytest.warns(RuntimeWarning, match="native half"), pytest.raises(ValueError, match="^q must"):
        binding.varlen_attn_fwd(q, q, q, torch.tensor([0, T]).int(), True, 0.1)
    with warnings.catch_warnings(), pytest.raises(ValueError, match="^o_parts must"):
        warnings.simplefilter("error")  # (said once)
        binding.varlen_attn_merge(q[None], q)
