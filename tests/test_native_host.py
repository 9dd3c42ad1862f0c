"""The native calls' object (csrc/bs_torch.cpp) without a GPU: who owns a stack's handle, and the buffers it keeps."""
import ctypes as C
import subprocess
import sys
import threading
import time

import pytest
import torch  # noqa: F401 (the native module links against it)

from paper_1804_08378_amd import _bs_torch
from paper_1804_08378_amd import brainslug as bs
from paper_1804_08378_amd import build
from paper_1804_08378_amd import workloads as wl

SHAPE = (2, 8, 12, 12)


class _Library:
    """The library with a destroy function that also counts."""

    def __init__(self, lib):
        self._lib, self.destroyed = lib, []
        self.bs_stack_destroy = C.CFUNCTYPE(None, C.c_void_p)(lambda h: self.destroyed.append(h))

    def __getattr__(self, name):
        return getattr(self._lib, name)


def _stack(layers=None, **opts):
    return bs.Stack(layers or [wl.bn_params(8, 1), wl.relu(), wl.maxpool(3, 2, 1)], SHAPE, "f32").plan(host_only=1, **opts)


def test_threads_that_ask_at_once_share_one_native_object(monkeypatch):
    """The object owns the handle: were two made, the one that is dropped would destroy it under the other."""
    lib = _Library(bs.load())
    monkeypatch.setattr(bs, "load", lambda: lib)
    made, real = [], _bs_torch.Plan

    def slow(*args):
        made.append(real(*args))
        time.sleep(0.2)  # every other thread gets to ask meanwhile
        return made[-1]

    monkeypatch.setattr(_bs_torch, "Plan", slow)
    st, got = _stack(), []
    threads = [threading.Thread(target=lambda: got.append(st.native())) for _ in range(4)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert len(made) == 1 and all(g is made[0] for g in got)
    handle = st.handle
    made.clear()
    got.clear()
    assert lib.destroyed == []
    del st
    assert lib.destroyed == [handle]
    lib._lib.bs_stack_destroy(handle)


def test_threads_that_need_the_backward_plan_at_once_plan_it_once(monkeypatch):
    """Planning again frees the plan that another thread may be running."""
    calls, real = [], bs.bs_stack_plan_backward

    def slow(handle):
        calls.append(handle)
        time.sleep(0.2)
        return real(handle)

    monkeypatch.setattr(bs, "bs_stack_plan_backward", slow)
    st = _stack()
    native, x = st.native(), torch.zeros(SHAPE)

    def first_call():
        with pytest.raises(Exception):  # no device: what is looked at is who plans
            st.backward(x, [], torch.zeros(1))

    threads = [threading.Thread(target=first_call) for _ in range(4)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert len(calls) == 1 and st._bwd_planned and st.native() is native
    st.plan_backward()  # asked for by name: planned anew
    assert len(calls) == 2
    st.close()


def test_python_and_native_calls_share_one_workspace():
    """Calls that go through Python (the first one, channel slices) and native ones on a stream use one buffer, forward and backward each."""
    st = _stack([wl.maxpool(3, 1, 1), wl.leaky_relu(0.1), wl.avgpool(2, 2), wl.relu(), wl.maxpool(3, 1, 1)], max_steps_per_sequence=1).plan_backward()
    assert st._workspace_bytes > 0 and st._bwd_workspace_bytes > 0
    for backward, n in ((False, st._workspace_bytes), (True, st._bwd_workspace_bytes)):
        a = st.workspace("cpu", 5, backward)
        assert a.numel() == n and a.data_ptr() == st.native().workspace(backward, torch.device("cpu"), 5).data_ptr()
        assert a.data_ptr() == st.workspace("cpu", 5, backward).data_ptr()
        other = st.native().workspace(backward, torch.device("cpu"), 6)  # another stream, asked for by a native call first
        assert other.data_ptr() != a.data_ptr() and st.workspace("cpu", 6, backward).data_ptr() == other.data_ptr()
    st.plan(host_only=1)  # one sequence: nothing to hand over, nothing kept
    assert st.workspace("cpu", 5) is None and not st._workspace and st.native().workspace(False, torch.device("cpu"), 5) is None
    st.close()


def test_nothing_is_allocated_while_another_thread_can_only_wait():
    """An allocation may call into the interpreter (here: a dispatch mode that lets other threads run).  A thread that then closes or plans the
    stack waits for the object with the interpreter's lock in its hand, so the allocation must not happen inside.  In a process of its own: the
    mistake is a deadlock."""
    code = """
import threading, time, torch
from torch.utils._python_dispatch import TorchDispatchMode
from paper_1804_08378_amd import brainslug as bs, workloads as wl
st = bs.Stack([wl.maxpool(3, 1, 1), wl.relu(), wl.maxpool(3, 1, 1)], (2, 8, 12, 12)).plan(host_only=1, max_steps_per_sequence=1)
inside = threading.Event()
class Slow(TorchDispatchMode):
    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        inside.set()
        time.sleep(0.5)
        return func(*args, **(kwargs or {}))
native = st.native()
def ask():
    with Slow():
        native.workspace(False, torch.device("cpu"), 3)
t = threading.Thread(target=ask)
t.start()
inside.wait()
st.close()
t.join()
print("done")
"""
    done = subprocess.run([sys.executable, "-c", code], cwd=bs.HERE + "/..", capture_output=True, text=True, timeout=90)
    assert done.stdout.strip().endswith("done"), done.stderr[-2000:]


def test_without_the_native_module_the_python_code_takes_every_call(monkeypatch):
    lib = _Library(bs.load())
    monkeypatch.setattr(bs, "load", lambda: lib)
    monkeypatch.setattr(bs, "_torch_module", None)
    monkeypatch.setattr(build, "TORCH_EXT", "/nonexistent/_bs_torch.so")
    st = _stack([wl.maxpool(3, 1, 1), wl.leaky_relu(0.1), wl.avgpool(2, 2), wl.relu(), wl.maxpool(3, 1, 1)], max_steps_per_sequence=1)
    with pytest.warns(RuntimeWarning, match="native calls"):
        n = st.native()
    assert n.run(None, []) is None and n.infer(None, []) is None and n.record(None, []) is None and n.backward(None, [], None, None) is None
    st.plan_backward()
    for backward, size in ((False, st._workspace_bytes), (True, st._bwd_workspace_bytes)):
        a = st.workspace("cpu", 5, backward)
        assert a.numel() == size and st.workspace("cpu", 5, backward) is a and st.workspace("cpu", 6, backward) is not a
    st.plan(host_only=1)
    assert st.workspace("cpu", 5) is None and st.native() is not n
    handle = st.handle
    del st
    assert lib.destroyed == [handle]
    lib._lib.bs_stack_destroy(handle)


def test_native_module_is_built_for_one_torch_and_optional(monkeypatch, tmp_path, capsys):
    assert build.torch_ext_fits() and build.up_to_date() and _bs_torch.built_for == build.torch_tag()
    with monkeypatch.context() as m:
        m.setattr(build, "torch_tag", lambda: "bs_torch for torch 0.0, none;")  # another torch than the file's
        assert not build.torch_ext_fits() and not build.up_to_date()
    with monkeypatch.context() as m:
        m.setattr(build, "torch_tag", lambda: "")  # no torch: the library alone
        assert build.up_to_date()
    stale = tmp_path / "_bs_torch.so"
    stale.write_bytes(b"older")
    monkeypatch.setattr(build, "TORCH_EXT", str(stale))
    monkeypatch.setenv("CXX", "false")
    assert build.try_torch_ext() is False and not stale.exists() and "without the native calls" in capsys.readouterr().err
