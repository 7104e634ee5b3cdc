"""A binding call without a stream runs on torch's current stream (GPU)."""
import pytest

pytestmark = pytest.mark.gpu


def test_default_stream_is_the_current_one():
    import torch

    from paper_2609_36760_amd import _binding as mb
    torch.zeros(1, device="cuda")
    side = torch.cuda.Stream()
    assert mb._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert mb._stream(None) == side.cuda_stream
    assert mb._stream(None) == torch.cuda.current_stream().cuda_stream
    assert mb._stream(side) == side.cuda_stream and mb._stream(side.cuda_stream) == side.cuda_stream
