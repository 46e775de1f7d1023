"""A launch without a stream goes on torch's current stream: the default one, a
side stream inside torch.cuda.stream(), and the default one again after it."""
import pytest
import torch

import paper_2509_17542_amd as K

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def test_default_stream_follows_torch():
    torch.zeros(1, device="cuda")
    default = torch.cuda.current_stream()
    assert K._stream(None) == default.cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert K._stream(None) == side.cuda_stream != default.cuda_stream
    assert K._stream(None) == default.cuda_stream
    assert K._stream(side) == side.cuda_stream
