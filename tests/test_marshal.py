"""The binding's extension module: what it refuses itself, and that statuses of the C ABI come through (no GPU: every
call here is refused before anything is launched)."""
import numpy as np
import pytest

import paper_1907_06154_amd.binding as b


def test_refusals_and_statuses():
    b.lib()
    m = b._fast
    f32, f64 = np.ones((3, 3), np.float32), np.ones((3, 3), np.float64)
    with pytest.raises(TypeError):
        m.conv2d(0, 0, 4, 4)
    with pytest.raises(TypeError):
        m.conv2d(None, 0, 4, 4, f32, -1, -1, 1, 0, 0)
    for bad, code in ((f64, 0), (f32, 1), (np.ones((3, 3, 3), np.float32), 0)):
        with pytest.raises(ValueError):
            m.conv2d(16, 1 << 20, 4, 4, bad, -1, -1, 1, code, 0)
    with pytest.raises((ValueError, BufferError)):
        m.stencil2d(16, 1 << 20, 4, 4, np.ones((6, 6), np.float32)[::2, ::2], 1, 0, 0)      # not contiguous
    assert m.conv2d(0, 1 << 20, 4, 4, f32, -1, -1, 1, 0, 0) == 1                             # null input
    assert m.conv2d(16, 1 << 20, 0, 4, f32, -1, -1, 1, 0, 0) == 2
    assert m.conv2d(16, 1 << 20, 4, 4, f32, 5, -1, 1, 0, 0) == 3
    assert m.conv3d(16, 1 << 20, 4, 4, 4, np.ones((3, 3, 3)), -1, -1, -1, 7, 1, 0) == 4
    assert m.stencil2d(16, 16, 4, 4, f32, 1, 0, 0) == 5
    assert m.stencil3d(16, 16, 4, 4, 4, np.ones((3, 3, 3)), 1, 1, 0) == 5
    assert m.iterate(16, 1 << 20, 4, 4, 1, f32, 1, 0, -1, 0)[0] == 3
    assert m.scan(16, 1 << 20, -1, 0, 0, 0, 0) == 2


def test_current_stream_without_the_private_query(monkeypatch):
    import types
    import torch
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1234))
    assert b._stream_ptr(None) == 1234
    assert b._stream_ptr(types.SimpleNamespace(cuda_stream=77)) == 77
