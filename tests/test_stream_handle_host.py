"""The binding takes torch's raw-handle functions where torch has them, and its public ones where it does not."""
import importlib.util
import types

import pytest

torch = pytest.importorskip("torch")


def test_without_the_private_functions(monkeypatch):
    from paper_2605_03109_amd import gsi

    for name in ("_cuda_getDevice", "_cuda_getCurrentRawStream"):
        monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: types.SimpleNamespace(cuda_stream=1000 + device))
    spec = importlib.util.spec_from_file_location("gsi_again", gsi.__file__)
    again = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(again)
    assert again._device() == 3 and again._stream() == 1003
    assert again._stream(types.SimpleNamespace(cuda_stream=7)) == 7
