"""The binding's host side without a GPU."""
import importlib.util
import os

import torch

import paper_2606_09794_amd as P


def _fresh_api():
    """A second copy of the binding's module, executed now."""
    path = os.path.join(os.path.dirname(P.__file__), "api.py")
    spec = importlib.util.spec_from_file_location(P.__name__ + "._api_copy", path)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_stream_query_without_the_private_entry_point(monkeypatch):
    """The stream comes from torch's public query where the raw one is missing."""
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.delattr(torch._C, "_cuda_getDevice", raising=False)

    class Stream:
        cuda_stream = 1234
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: Stream)
    assert _fresh_api()._stream() == 1234


def test_stream_query_initialises_the_device(monkeypatch):
    """The raw query is asked for the device that torch's public call names, which
    initialises the GPU where nothing has yet."""
    asked = []
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: asked.append(d) or 99, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert _fresh_api()._stream() == 99 and asked == [3]
