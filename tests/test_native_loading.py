"""First use of the binding where the native module cannot be loaded, and where two threads meet in it (no GPU needed)."""
import ctypes
import threading
import types

import pytest
import torch

from paper_2411_19419_amd import binding


@pytest.fixture
def unloaded(monkeypatch):
    """The binding as it is before its first call that needs torch."""
    for name in ("_raw_stream", "_current_device", "_native"):
        monkeypatch.setattr(binding, name, None)
    monkeypatch.setattr(binding, "torch", binding._Torch())
    return monkeypatch


def _fails():
    raise ImportError("undefined symbol")


def test_without_the_native_module_every_call_takes_ctypes(unloaded):
    unloaded.setattr(binding, "_load_native", _fails)
    with pytest.warns(RuntimeWarning, match="undefined symbol"):
        assert binding.torch.float32 is torch.float32
    assert binding.torch is torch and binding._native is None
    assert binding._raw_stream is not None and binding._current_device is not None

    called = []

    class Library:
        def __getattr__(self, name):
            return lambda *args: called.append(name) or 0

    unloaded.setattr(binding, "_load", Library)
    unloaded.setattr(binding, "_raw_stream", lambda index: 0)
    unloaded.setattr(binding, "_current_device", lambda: 0)
    unloaded.setattr(binding, "_default_stream", lambda device: None)
    multi = object.__new__(binding.ConvMulti)
    multi._handle, multi.ys = ctypes.c_void_p(8), ["y"]
    assert multi.apply() == ["y"] and called == ["conv_multi_apply"]
    multi._handle = None
    kernel = types.SimpleNamespace(device=types.SimpleNamespace(index=0), record_stream=lambda stream: called.append("recorded"))
    plan = binding.ConvPlan(ctypes.c_void_p(8), (1, 1, 1, 1, 0), (1, 1), 1, None, None, None, kernel)
    plan.close()
    assert plan._handle is None and called[1:] == ["recorded", "conv_plan_destroy"]


def test_a_second_thread_sees_all_or_nothing(unloaded):
    loading, go_on = threading.Event(), threading.Event()
    native = object()

    def slow():
        loading.set()
        assert go_on.wait(30)
        return native

    unloaded.setattr(binding, "_load_native", slow)
    seen = []

    def use():
        binding.torch.float32
        seen.append((binding._native, binding._raw_stream is not None, binding.torch is torch))

    first, second = threading.Thread(target=use), threading.Thread(target=use)
    first.start()
    assert loading.wait(30)
    second.start()
    second.join(0.2)
    assert second.is_alive() and binding.torch is not torch      # (waits for the first one's loading)
    go_on.set()
    for t in (first, second):
        t.join(30)
    assert seen == [(native, True, True)] * 2
