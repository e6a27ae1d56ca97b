"""The binding hands the library torch's current stream, whichever way it was made current."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_binding_follows_the_current_stream():
    from paper_2405_16528_amd import binding as L
    assert L._stream() == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert L._stream() == side.cuda_stream
        with torch.cuda.stream(torch.cuda.default_stream()):
            assert L._stream() == torch.cuda.default_stream().cuda_stream
        assert L._stream() == side.cuda_stream
    torch.cuda.set_stream(side)
    try:
        assert L._stream() == side.cuda_stream
    finally:
        torch.cuda.set_stream(torch.cuda.default_stream())
    assert L._stream() == torch.cuda.current_stream().cuda_stream
