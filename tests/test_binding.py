"""What the Python side itself promises: types of arrays at the bare library, the stream without torch's private helpers."""
import ctypes as C
import importlib
import types

import numpy as np
import pytest

from paper_2510_25412_amd import binding


def test_bare_library_refuses_arrays_of_another_type():
    ctx = binding.Context(binding.make_config(32, 8, 128, 16, "bf16", 8, device=-1))
    f = ctx.kv_open(None)
    kv, wrong = np.array([f], np.int32), np.array([f], np.int64)
    length = np.zeros(1, np.int64)
    p32, p64 = C.POINTER(C.c_int32), C.POINTER(C.c_int64)
    assert ctx.lib is binding.load()
    assert ctx.lib.sym_kv_truncate(ctx.h, 1, binding.as_i32p(kv), length.ctypes.data_as(p64)) == 0
    for bad in (wrong.ctypes.data_as(p64), kv.ctypes.data, C.c_void_p(kv.ctypes.data)):
        with pytest.raises(C.ArgumentError):
            ctx.lib.sym_kv_truncate(ctx.h, 1, bad, length.ctypes.data_as(p64))
    with pytest.raises(C.ArgumentError):
        ctx.lib.sym_kv_truncate(ctx.h, 1, kv.ctypes.data_as(p32), kv.ctypes.data_as(p32))
    ctx.kv_truncate(wrong, [0])                   # the methods convert
    assert ctx.kv_pages(f) == [] and ctx.last_moves().shape == (0, 2)


def test_stream_without_the_private_name(monkeypatch):
    torch = pytest.importorskip("torch")
    from paper_2510_25412_amd import driver
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device: types.SimpleNamespace(cuda_stream=(str(device), 7)))
    try:
        importlib.reload(driver)
        sess = driver.HipSession.__new__(driver.HipSession)
        sess.device = torch.device("cuda:0")
        assert sess.stream == ("cuda:0", 7)
    finally:
        monkeypatch.undo()
        importlib.reload(driver)
