"""GPU tests of the binding's stream lookups, by ctypes and by the native module: a call without a stream goes to the current one."""
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


def test_the_module_finds_the_current_stream(device):
    """A call without a stream comes after the work that the current stream has, and before what follows it there."""
    pkv.lib()
    assert not isinstance(pkv._call, pkv._ByCtypes)   # as built, it is there
    shape = pkv.make_shape(1, 8, 8, 1, 1, 128)
    tables, lens = torch.zeros(1, 1, dtype=torch.int32, device=device), torch.ones(1, dtype=torch.int32, device=device)
    new = torch.arange(1, 1025, dtype=torch.int16, device=device)
    x = torch.randn(4096, 4096, device=device)
    y = torch.mm(x, x)
    for stream in (torch.cuda.Stream(), torch.cuda.default_stream(), torch.cuda.Stream()):
        row = torch.zeros_like(new)
        pools = [torch.zeros(1, 8, 16, 128, dtype=torch.int16, device=device) for _ in range(2)]
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            for _ in range(30):
                torch.mm(x, x, out=y)     # some ms
            row.copy_(new)
            pkv.kv_append(row, row, *pools, tables, lens, shape)
            row.zero_()
        stream.synchronize()
        for pool in pools:
            assert torch.equal(pool[0, :, 0].reshape(-1), new) and not pool[0, :, 1:].any()
