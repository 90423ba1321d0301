"""Calls go to the stream that torch calls current: the default one, another one, one under capture."""
import pytest
import torch

from paper_2505_11157_amd import binding

pytestmark = pytest.mark.gpu


def test_stream_is_the_current_one():
    x = torch.zeros(1, device="cuda:0")
    raw = lambda: binding._stream().value or 0
    assert raw() == torch.cuda.current_stream().cuda_stream
    other = torch.cuda.Stream()
    with torch.cuda.stream(other):
        assert raw() == other.cuda_stream
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert raw() == torch.cuda.current_stream().cuda_stream
        x.add_(1)
    assert raw() == torch.cuda.current_stream().cuda_stream
    torch.cuda.synchronize()
