"""Calls without a stream argument go to torch's current stream: the default one, a stream of a `with` block, and the
stream of a graph under capture."""
import pytest
import torch

from paper_1706_08359_amd import binding as B

pytestmark = pytest.mark.gpu


def test_handle_is_that_of_the_current_stream():
    print("current stream", flush=True)
    assert B._stream(None) == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert B._stream(None) == side.cuda_stream == B._stream(side)
    assert B._stream(None) == torch.cuda.current_stream().cuda_stream
    graph, x = torch.cuda.CUDAGraph(), torch.zeros(4, device="cuda")
    with torch.cuda.graph(graph):
        seen, own = B._stream(None), torch.cuda.current_stream().cuda_stream
        x.add_(1)
    assert seen == own
