"""A call without a stream goes to torch's current stream."""
import pytest

from paper_2609_10018_amd import ffi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_default_stream_is_the_current_one():
    assert ffi._stream_ptr(None) == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert ffi._stream_ptr(None) == side.cuda_stream
    assert ffi._stream_ptr(None) == torch.cuda.current_stream().cuda_stream
    assert ffi._stream_ptr(side) == side.cuda_stream
    assert ffi._stream_ptr(side.cuda_stream) == side.cuda_stream
