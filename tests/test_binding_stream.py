"""The stream handle that the binding passes."""
from types import SimpleNamespace

import pytest
import torch

import paper_2001_04931_amd.binding as B


def test_public_call_where_torch_lacks_the_raw_handle(monkeypatch):
    """torch's accessor of the raw handle is private: without it every entry point
    takes the handle of the public Stream object."""
    monkeypatch.setattr(B, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=1234))
    assert B._stream() == 1234
    assert B._stream(SimpleNamespace(cuda_stream=77)) == 77


@pytest.mark.gpu
def test_both_ways_name_the_current_stream(monkeypatch):
    side = torch.cuda.Stream()
    for s in (torch.cuda.current_stream(), side):
        with torch.cuda.stream(s):
            assert B._stream() == s.cuda_stream
            with monkeypatch.context() as m:
                m.setattr(B, "_raw_stream", None)
                assert B._stream() == s.cuda_stream
