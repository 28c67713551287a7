"""Work goes to torch's current stream of the current device."""
import pytest
import torch

from paper_2304_04237_amd import binding

pytestmark = pytest.mark.gpu


def test_current_stream_handle():
    assert binding._stream() == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert binding._stream() == side.cuda_stream
    assert binding._stream() == torch.cuda.current_stream().cuda_stream != side.cuda_stream
