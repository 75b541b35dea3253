"""The stream that the binding passes when none is given.  (Not the first of the GPU tests: the demo in C is started while nothing drives the GPU yet.)"""
import importlib.util

import pytest
import torch

from paper_2501_10054_amd import tardis as T


class _Stream:
    cuda_stream = 4096


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_without_the_private_names(monkeypatch, missing):
    """They are no part of torch's interface: without them the public call serves."""
    monkeypatch.setattr(torch.cuda, "current_stream", _Stream)
    monkeypatch.delattr(torch._C, missing, raising=False)
    spec = importlib.util.spec_from_file_location("another_tardis", T.__file__)
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    assert module._stream(None).value == 4096


@pytest.mark.gpu
def test_it_is_the_current_stream():
    assert (T._stream(None).value or 0) == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert T._stream(None).value == torch.cuda.current_stream().cuda_stream == s.cuda_stream
    assert T._stream(s).value == s.cuda_stream
