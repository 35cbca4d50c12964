"""A call without a stream goes to the current one, on the default stream, inside a stream context and after it."""
import pytest

pytestmark = pytest.mark.gpu


def test_default_stream_is_the_current_one():
    import torch

    from paper_2503_12211_amd import binding
    side = torch.cuda.Stream()
    assert binding._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert binding._stream(None) == side.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert binding._stream(None) == torch.cuda.current_stream().cuda_stream != side.cuda_stream
    assert binding._stream(side) == binding._stream(side.cuda_stream) == side.cuda_stream
