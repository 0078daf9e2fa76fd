"""The stream that the binding passes to the library: the caller's current one,
through torch's raw handle or, in a torch without it, the public call.
"""
import types

import pytest
import torch

import paper_1705_07272_amd as rrt


def test_without_the_raw_handle(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(rrt, "_raw_stream", None, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=4096))
    assert rrt._stream().value == 4096


@pytest.mark.gpu
@pytest.mark.parametrize("raw", [True, False])
def test_current_stream(monkeypatch, raw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if not raw:
        monkeypatch.setattr(rrt, "_raw_stream", None)
    assert (rrt._stream().value or 0) == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert rrt._stream().value == s.cuda_stream
