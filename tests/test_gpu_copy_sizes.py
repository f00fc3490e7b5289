"""GPU test of the block copies at the edges of their slices (256 chunks of 16 bytes): blocks of a part of a
slice, of whole slices, of odd numbers of chunks, short lists, ids outside the pool."""
import pytest
import torch

from paper_2602_11530_amd import binding as pkv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block_bytes", [16, 48, 2048, 4080, 4096, 4112, 8192, 12288, 12304, 20480, 65536])
@pytest.mark.parametrize("n", [1, 3, 64, 257])
@pytest.mark.expects_id_faults
def test_slices(device, block_bytes, n, id_faults):
    g = torch.Generator(device=device)
    g.manual_seed(block_bytes * 1000 + n)
    pool_blocks = 2 * n + 3
    pools = [torch.randint(0, 256, (pool_blocks, block_bytes), dtype=torch.uint8, device=device, generator=g) for _ in range(2)]
    ids = [torch.randperm(pool_blocks, device=device, generator=g).to(torch.int32)[:n].contiguous() for _ in range(2)]
    ids[0][n // 2] = pool_blocks   # never followed
    keep = torch.arange(n, device=device) != n // 2
    a, b = ids[0][keep].long(), ids[1][keep].long()
    src, dst = pools
    staging = torch.full((n, block_bytes), 7, dtype=torch.uint8, device=device)
    want = staging.clone()
    want[keep] = src[a]
    pkv.kv_blocks_gather(src, ids[0], staging, n, block_bytes, pool_blocks)
    assert torch.equal(staging, want)
    want = dst.clone()
    want[b] = src[a]
    moved = dst.clone()
    pkv.kv_blocks_move(src, ids[0], moved, ids[1], n, block_bytes, pool_blocks, pool_blocks)
    assert torch.equal(moved, want)
    want = dst.clone()
    want[a] = staging[keep]
    pkv.kv_blocks_scatter(staging, dst, ids[0], n, block_bytes, pool_blocks)
    assert torch.equal(dst, want)
    torch.cuda.synchronize()
    assert int(id_faults.item()) == 3
    id_faults.zero_()


@pytest.mark.parametrize("block_bytes,n", [
    (8192, 511), (8192, 512), (8192, 513), (24576, 171),            # two chunks per lane from 4 MB on, in blocks of 8 and 24 KiB
    (16384, 4095), (16384, 4096), (49152, 1366), (65536, 1025),     # and in a scatter from 64 MB on
    (12288, 5462),                                                  # neither
])
@pytest.mark.expects_id_faults
def test_chunks_per_lane(device, block_bytes, n, id_faults):
    g = torch.Generator(device=device)
    g.manual_seed(block_bytes + n)
    pool_blocks = n + 3
    src, dst = [torch.randint(0, 256, (pool_blocks, block_bytes), dtype=torch.uint8, device=device, generator=g) for _ in range(2)]
    ids = torch.randperm(pool_blocks, device=device, generator=g).to(torch.int32)[:n].contiguous()
    ids[n // 2] = -1   # never followed
    keep = torch.arange(n, device=device) != n // 2
    staging = torch.full((n + 1, block_bytes), 7, dtype=torch.uint8, device=device)
    want = staging.clone()
    want[:n][keep] = src[ids[keep].long()]
    pkv.kv_blocks_gather(src, ids, staging, n, block_bytes, pool_blocks)
    assert torch.equal(staging, want)
    want = dst.clone()
    want[ids[keep].long()] = staging[:n][keep]
    pkv.kv_blocks_scatter(staging, dst, ids, n, block_bytes, pool_blocks)
    assert torch.equal(dst, want)
    torch.cuda.synchronize()
    assert int(id_faults.item()) == 2
    id_faults.zero_()
