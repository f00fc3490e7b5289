"""GPU test of the binding's stream lookup: a call without a stream goes to the current one."""
import pytest
import torch

from paper_2602_11530_amd import binding as pkv

pytestmark = pytest.mark.gpu


def test_default_is_the_current_stream(device):
    pkv.lib()
    assert pkv._stream(None) == (torch.cuda.current_stream().cuda_stream or None)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert pkv._stream(None) == side.cuda_stream
        with torch.cuda.stream(torch.cuda.default_stream()):
            assert pkv._stream(None) == (torch.cuda.default_stream().cuda_stream or None)
        assert pkv._stream(None) == side.cuda_stream
    assert pkv._stream(side) == pkv._stream(side.cuda_stream) == side.cuda_stream
