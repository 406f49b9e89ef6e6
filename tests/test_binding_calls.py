"""The native device calls of Context convert their arguments as the ctypes signatures of the C ABI do.  No GPU:
the entry points are stood in for by a function that writes down what arrives."""
import ctypes as C
import inspect
import os
import subprocess
import sys
import typing

import numpy as np
import pytest

import paper_1912_09268_amd as M
from paper_1912_09268_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CALLS = {
    "pack": ["group", "d_grad_ptrs", "d_merge_bufs"],
    "pack_tensors": ["first_tensor", "last_tensor", "d_grad_ptrs", "d_merge_bufs"],
    "reduce": ["group", "d_merge_bufs", "d_reduced"],
    "unpack_update": ["group", "d_reduced", "d_w_ptrs", "d_v_ptrs", "lr", "momentum"],
    "reduce_update": ["group", "d_merge_bufs", "d_w_ptrs", "d_v_ptrs", "lr", "momentum"],
    "group_pipeline": ["group", "d_grad_ptrs", "d_merge_bufs", "d_reduced", "d_w_ptrs", "d_v_ptrs", "lr", "momentum"],
    "direct_update": ["group", "d_grad_ptrs", "d_reduced", "d_w_ptrs", "d_v_ptrs", "lr", "momentum"],
    "group_pipeline_span": ["group_first", "group_count", "d_grad_ptrs", "d_merge_bufs", "d_reduced", "d_w_ptrs",
                            "d_v_ptrs", "lr", "momentum"],
    "group_pipeline_static": ["group", "d_grad_ptrs", "d_merge_bufs", "d_reduced", "d_w_ptrs", "d_v_ptrs", "lr", "momentum"],
}


@pytest.fixture
def recorder():
    """Entry points that keep their arguments, and the real ones again afterwards."""
    from paper_1912_09268_amd import _calls
    real = {name: C.cast(getattr(M.lib(), name), C.c_void_p).value for name in binding._SIGNATURES}
    seen, keep, table = [], [], dict(real)
    status = [0]
    for name in CALLS:
        types = binding._SIGNATURES["mgwfbp_" + name][1]

        def record(*args, name=name):
            seen.append((name, args))
            return status[0]

        fn = C.CFUNCTYPE(C.c_int, *types)(record)
        keep.append(fn)
        table["mgwfbp_" + name] = C.cast(fn, C.c_void_p).value
    _calls.set_functions(binding._check, table)
    yield seen, status
    _calls.set_functions(binding._check, real)


def _values(names):
    return {n: 0.1 * (k + 1) if n in ("lr", "momentum") else (k + 2 if not n.startswith("d_") else (0x7F00 << 32) + 64 * k)
            for k, n in enumerate(names)}


@pytest.mark.parametrize("name", sorted(CALLS))
def test_arguments_arrive_as_given(name, recorder):
    seen, _ = recorder
    ctx = M.Context([10, 20], [0, 1], 2, M.F32, host_only=True)
    names = CALLS[name]
    values = _values(names)
    want = tuple(float(np.float32(v)) if isinstance(v, float) else v for v in values.values())
    call = getattr(ctx, name)
    call(*values.values())
    call(*values.values(), 99)
    call(stream=99, **values)
    call(*list(values.values())[:2], **{n: values[n] for n in names[2:]}, stream=99)
    for k, (got_name, got) in enumerate(seen):
        assert got_name == name
        assert got == (ctx._h.value, *want, None if k == 0 else 99)
    ctx.close()
    call(*values.values())
    assert seen[-1][1][0] is None            # a closed context is a null pointer to the library


def test_odd_arguments(recorder):
    seen, _ = recorder
    ctx = M.Context([10], [0], 1, M.F32, host_only=True)
    ctx.pack(np.int64(-1), None, True, None)                 # int() for integers, None and bool as ctypes takes them
    assert seen[-1][1] == (ctx._h.value, -1, None, 1, None)
    ctx.pack((1 << 32) + 3, (1 << 64) - 8, 5)                # kept to the type's bits, as ctypes does
    assert seen[-1][1] == (ctx._h.value, 3, (1 << 64) - 8, 5, None)
    ctx.group_pipeline(0, 1, 2, 0, 3, 4, 1, np.float64(0.5))
    assert seen[-1][1] == (ctx._h.value, 0, 1, 2, None, 3, 4, 1.0, 0.5, None)
    n = len(seen)
    for bad in ((), (0, 1), (0, 1, 2, 3, 4), ("x", 1, 2), (0, 1.5, 2), (0, "a", 2), (None, 1, 2), (0, np.int64(4), 2)):
        with pytest.raises((TypeError, ValueError)):
            ctx.pack(*bad)
    for bad in ({"group": 0}, {"grop": 0}):
        with pytest.raises(TypeError):
            ctx.pack(0, 1, 2, **bad)
    with pytest.raises((TypeError, ValueError)):
        ctx.reduce_update(0, 1, 2, 3, "fast", 0.9)
    assert len(seen) == n
    ctx.close()


def test_a_failed_call_raises_with_its_status(recorder):
    _, status = recorder
    ctx = M.Context([10], [0], 1, M.F32, host_only=True)
    status[0] = -4
    with pytest.raises(M.MgwfbpError) as e:
        ctx.group_pipeline_static(0, 1, 2, 0, 3, 4, 0.1, 0.9)
    assert e.value.status == -4 and "mgwfbp_group_pipeline_static failed: MGWFBP_ECAPACITY" in str(e.value)
    ctx.close()


def test_subclasses_override_device_calls():
    class Counting(M.Context):
        calls = 0

        def pack(self, *args):
            self.calls += 1
            return super().pack(*args)

    ctx = Counting([10], [0], 1, M.F32, host_only=True)
    with pytest.raises(M.MgwfbpError):
        ctx.pack(0, 1, 2)                    # a host-only context: the library refuses
    assert ctx.calls == 1
    ctx.close()


def _in_a_fresh_interpreter(code):
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return r.stdout


def test_without_the_extension_module_everything_goes_through_ctypes():
    """No module for this Python: planning, contexts and device calls work as they do with it."""
    out = _in_a_fresh_interpreter("""
import sys
sys.modules["paper_1912_09268_amd._calls"] = None          # importing it raises ImportError
import paper_1912_09268_amd as M
merged, groups = M.plan([4, 4000, 4], [1e-3] * 3, 1e-2, 1e-9)
ctx = M.Context([1, 1000, 1], merged, 2, M.F32, host_only=True)
try:
    ctx.group_pipeline(0, 1, 2, 0, 3, 4, 0.1, 0.9)
except M.MgwfbpError as e:
    print(len(merged), e.status, type(M.Context.pack).__name__)
""")
    assert out.split() == ["3", "-1", "function"]


def test_device_calls_are_methods_from_the_start_and_stay_as_patched():
    """What is put in place of a device call before the library is loaded is still there afterwards."""
    out = _in_a_fresh_interpreter("""
import paper_1912_09268_amd as M
real = M.Context.pack
def counting(self, *args):
    print("counted", args)
    return real(self, *args)
M.Context.pack = counting
ctx = M.Context([4], [0], 1, M.F32, host_only=True)
try:
    ctx.pack(0, 1, 2)
except M.MgwfbpError as e:
    print(e.status, M.Context.pack is counting)
""")
    assert out.splitlines() == ["counted (0, 1, 2)", "-1 True"]


@pytest.mark.parametrize("name", sorted(CALLS))
def test_signatures_and_hints(name):
    call = getattr(M.Context, name)
    sig = inspect.signature(call)
    assert list(sig.parameters) == ["self", *CALLS[name], "stream"] and sig.parameters["stream"].default == 0
    hints = typing.get_type_hints(call)
    assert hints.pop("return") is type(None)
    assert hints == {n: float if n in ("lr", "momentum") else int for n in CALLS[name] + ["stream"]}
    assert call.__name__ == name and call.__qualname__ == f"Context.{name}" and call.__module__ == binding.__name__
    ctx = M.Context([10], [0], 1, M.F32, host_only=True)
    assert list(inspect.signature(getattr(ctx, name)).parameters) == [*CALLS[name], "stream"]
    ctx.close()


def test_a_replaced_entry_point_is_the_one_called(monkeypatch):
    ctx = M.Context([10], [0], 1, M.F32, host_only=True)
    seen = []
    with monkeypatch.context() as m:
        m.setattr(M.lib(), "mgwfbp_pack", lambda *args: seen.append(args) or 0)
        ctx.pack(0, 1, 2)
        assert len(seen) == 1 and seen[0][1] == 0 and seen[0][2].value == 1
        with pytest.raises(M.MgwfbpError):
            ctx.reduce(0, 1, 2)                  # the others are the library's
    with pytest.raises(M.MgwfbpError):
        ctx.pack(0, 1, 2)                        # and this one again
    assert len(seen) == 1
    ctx.close()


def test_a_call_keeps_no_reference():
    ctx = M.Context([10], [0], 1, M.F32, host_only=True)
    before = sys.getrefcount(ctx)
    bound = ctx.pack
    for _ in range(100):
        with pytest.raises(M.MgwfbpError):
            bound(0, 1, 2)
        with pytest.raises(TypeError):
            ctx.pack(0, "a", 2)
        with pytest.raises(AttributeError):
            M.Context.pack(object(), 0, 1, 2)    # no context at all
    del bound
    assert sys.getrefcount(ctx) == before
    ctx.close()
