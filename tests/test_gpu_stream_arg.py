"""The binding enqueues on torch's current stream (the default one, another one made current,
a stream under graph capture) or on the stream passed to it."""
import pytest
import torch

from paper_2002_04013_amd import abi

pytestmark = pytest.mark.gpu


def test_current_stream_handle():
    assert abi._stream().value == (torch.cuda.current_stream().cuda_stream or None)
    s, t = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert abi._stream().value == s.cuda_stream == torch.cuda.current_stream().cuda_stream
        with torch.cuda.stream(t):
            assert abi._stream().value == t.cuda_stream
        assert abi._stream().value == s.cuda_stream
        assert abi._stream(t).value == t.cuda_stream
    x = torch.zeros(4, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        x.add_(1)
        assert abi._stream().value == torch.cuda.current_stream().cuda_stream
    g.replay()
    torch.cuda.synchronize()
    assert bool((x == 1).all())
