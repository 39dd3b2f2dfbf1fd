"""The binding launches on the stream that is current where it is called."""
import pytest

pytestmark = pytest.mark.gpu


def test_current_stream_handle():
    import torch
    from paper_2605_29843_amd import harp
    side = torch.cuda.Stream()
    assert harp._stream_ptr(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert harp._stream_ptr(None) == side.cuda_stream
    assert harp._stream_ptr(side) == side.cuda_stream
    assert harp._stream_ptr(None) == torch.cuda.current_stream().cuda_stream
