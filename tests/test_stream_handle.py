"""The handle of the current stream comes from two functions of torch that are not
part of its interface, or, where a release lacks them, from the Stream object."""
import types

import pytest

from paper_2007_10752_amd import tdes as T


@pytest.mark.parametrize("missing", [None, "_cuda_getCurrentRawStream", "_cuda_getDevice"])
@pytest.mark.parametrize("initialized", [True, False])
def test_current_stream_with_and_without_the_raw_functions(monkeypatch, missing, initialized):
    import torch
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: initialized)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1234))
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 5000 + device,
                        raising=False)
    if missing:
        monkeypatch.delattr(torch._C, missing)
    want = 5003 if initialized and missing is None else 1234
    assert T._stream_handle(None) == want
    assert T._stream_handle(types.SimpleNamespace(cuda_stream=77)) == 77
