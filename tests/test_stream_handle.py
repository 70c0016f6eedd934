"""The stream that calls are enqueued on: the current one, whether or not torch has the function that gives its handle directly."""
import types

import pytest
import torch

from paper_2502_01703_amd import binding as Q


def test_without_the_raw_handle(monkeypatch):
    monkeypatch.setattr(Q, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    assert Q._stream() == 77


@pytest.mark.gpu
def test_both_ways_name_the_current_stream(monkeypatch):
    print("[case] stream handles", flush=True)
    side = torch.cuda.Stream()
    raw = [Q._stream()]
    with torch.cuda.stream(side):
        raw.append(Q._stream())
    assert raw == [torch.cuda.current_stream().cuda_stream, side.cuda_stream]
    monkeypatch.setattr(Q, "_raw_stream", None)
    P = torch.randn(5, 128, device="cuda")
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        assert Q._stream() == side.cuda_stream
        codes = Q.quantize(P, 4)[0]
    torch.cuda.current_stream().wait_stream(side)
    assert torch.equal(codes, Q.quantize(P, 4)[0])
