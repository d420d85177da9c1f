"""Calls without a stream run on torch's current one: the default stream, and one that a program has switched to."""
import pytest

from paper_2305_12213_amd import binding

pytestmark = pytest.mark.gpu


def test_current_stream_of_torch():
    import torch
    torch.cuda.init()
    other = torch.cuda.Stream()
    assert binding._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(other):
        assert binding._stream(None) == other.cuda_stream
        g, p = torch.ones(1024, device="cuda"), torch.zeros(1024, device="cuda")
        binding.sgd_update(p, g, 1024, 0.5)
        assert bool((p == -0.5).all())
    assert binding._stream(None) == torch.cuda.current_stream().cuda_stream != other.cuda_stream
    assert binding._stream(17) == 17
