"""The stream that a call without one goes to is torch's current stream, whichever that is."""
import pytest
import torch

from paper_1805_08768_amd import binding as sbc

pytestmark = pytest.mark.gpu


def test_calls_without_a_stream_take_the_current_one():
    assert (sbc._stream_handle(None).value or 0) == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert sbc._stream_handle(None).value == s.cuda_stream
        with torch.cuda.stream(torch.cuda.default_stream()):
            assert (sbc._stream_handle(None).value or 0) == torch.cuda.default_stream().cuda_stream
        assert sbc._stream_handle(None).value == s.cuda_stream
    assert sbc._stream_handle(s).value == s.cuda_stream and sbc._stream_handle(s.cuda_stream).value == s.cuda_stream
