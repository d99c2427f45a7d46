"""The binding's default stream is torch's current one: default stream, a side stream, one inside another, a capture."""
import pytest
import torch

from paper_2502_11058_amd import binding as B

pytestmark = pytest.mark.gpu


def test_current_stream_follows_torch():
    assert torch.cuda.is_available(), "no GPU visible"
    same = lambda: B._stream_handle(None) == torch.cuda.current_stream().cuda_stream  # noqa: E731
    assert same() and same()
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(a):
        assert B._stream_handle(None) == a.cuda_stream
        with torch.cuda.stream(b):
            assert B._stream_handle(None) == b.cuda_stream
        assert B._stream_handle(None) == a.cuda_stream
    assert same() and B._stream_handle(a) == a.cuda_stream and B._stream_handle(7) == 7
    x = torch.zeros(4, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        assert same()
        x.add_(1.0)
    assert same()
