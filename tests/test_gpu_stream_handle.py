"""The binding's stream argument: the handle it passes on is the current stream's, or the
given one's, whether or not torch hands out raw handles."""
import pytest
import torch

from paper_2606_03928_amd import vase

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("device", [DEV, torch.device("cuda")])
def test_stream_handle(monkeypatch, device):
    side = torch.cuda.Stream(DEV)

    def check():
        assert vase._stream_ptr(device, side) == side.cuda_stream
        assert vase._stream_ptr(device, None) == torch.cuda.current_stream(DEV).cuda_stream
        with torch.cuda.stream(side):
            assert vase._stream_ptr(device, None) == side.cuda_stream

    check()
    monkeypatch.setattr(vase, "_raw_stream", None)
    check()
