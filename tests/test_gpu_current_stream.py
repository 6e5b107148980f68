"""Calls go to torch's current stream of the current device, or to the stream that is passed."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_stream_handle():
    from paper_2605_03109_amd import gsi

    assert gsi._device() == torch.cuda.current_device()
    assert gsi._stream() == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert gsi._stream() == s.cuda_stream
        assert gsi._stream(torch.cuda.default_stream()) == torch.cuda.default_stream().cuda_stream
    assert gsi._stream(s) == s.cuda_stream
    assert gsi._stream() == torch.cuda.current_stream().cuda_stream
