"""The handle the calls enqueue on is the current torch stream's, for a device with
and without an index."""
import pytest

from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


def test_stream_handle_follows_the_current_stream():
    require_gpu()
    import torch
    from paper_2606_21410_amd.api import _stream_handle
    side = torch.cuda.Stream()
    for dev in (torch.device("cuda"), torch.device("cuda", torch.cuda.current_device())):
        assert _stream_handle(dev) == torch.cuda.current_stream().cuda_stream
        with torch.cuda.stream(side):
            assert _stream_handle(dev) == side.cuda_stream != torch.cuda.default_stream().cuda_stream
        assert _stream_handle(dev) == torch.cuda.current_stream().cuda_stream
