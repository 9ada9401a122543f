"""The binding's current stream, with and without torch's internal call for its handle."""
import importlib.util
import types

import pytest

torch = pytest.importorskip("torch")

from paper_2608_11231_amd import lkv  # noqa: E402


def _fresh_binding():
    spec = importlib.util.spec_from_file_location("lkv_fresh", lkv.__file__)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_stream_without_the_internal_call(missing, monkeypatch):
    monkeypatch.delattr(torch._C, missing, raising=False)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=4711))
    assert _fresh_binding()._stream(None) == 4711


def test_stream_with_it(monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda dev: 100 + dev, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    assert _fresh_binding()._stream(None) == 103


def test_given_streams():
    assert lkv._stream(types.SimpleNamespace(cuda_stream=9)) == 9 and lkv._stream(12) == 12
