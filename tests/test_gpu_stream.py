"""A call without a stream goes to torch's current stream, whichever that is."""

import pytest
import torch

from paper_2509_00195_amd import tts

pytestmark = pytest.mark.gpu


def test_default_stream_follows_torch():
    torch.zeros(1, device="cuda")
    side = torch.cuda.Stream()
    assert tts._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert tts._stream(None) == side.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert tts._stream(None) == torch.cuda.current_stream().cuda_stream
    assert tts._stream(side) == side.cuda_stream and tts._stream(7) == 7
