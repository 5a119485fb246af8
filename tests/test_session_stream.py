"""Session.stream is torch's current stream, also under a torch without the two
private functions that give its handle directly."""
import types

import pytest
import torch

from paper_2605_20600_amd.session import Session


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_stream_without_the_private_functions(monkeypatch, missing):
    monkeypatch.delattr(torch._C, missing, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda: types.SimpleNamespace(cuda_stream=77))
    assert Session.stream() == 77


@pytest.mark.gpu
def test_stream_is_the_current_one():
    assert Session.stream() == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert Session.stream() == s.cuda_stream
    assert Session.stream() == torch.cuda.current_stream().cuda_stream
