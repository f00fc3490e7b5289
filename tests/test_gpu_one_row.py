"""GPU parity of batches of 32 to 64 segments (request, KV head) of one row of 64 floats each: with fewer blocks than wavefronts, as many
and more, a few blocks each and up to thousands; the bounds tight and wide, which changes no bit; batches that turn out on the device
to be cut along their segments; replays that go from one to the other."""
import numpy as np
import pytest
import torch

import oracle
import routes
from gpu_util import REL_L2, abs_error_within_bar, run_attn_dev, shape_of, to_bits, to_dev
from paper_2602_11530_amd import binding as pkv
from paper_2602_11530_amd import workloads as wl
from test_gpu_fp8kv import KS, VS, check as check_fp8, run_fp8

pytestmark = pytest.mark.gpu


def spread(total, n, longest, empty=0):
    """n lengths of `total` blocks together, the first of `longest`, the last `empty` of none, not all of them whole blocks."""
    rest = n - 1 - empty
    each = [(total - longest) // rest + (i < (total - longest) % rest) for i in range(rest)]
    lens = [16 * longest] + [max(16 * b - 5 * i % 16, 1) if b else 0 for i, b in enumerate(each)] + [0] * empty
    assert len(lens) == n and sum((x + 15) // 16 for x in lens) == total and max(lens) == 16 * longest
    return lens


# lengths, heads, blocks that the table has room for, what becomes of it
BATCHES = [
    (spread(255, 32, 50), 1, 50, "records"),           # a block in all but one of the workgroups
    (spread(600, 40, 60, 3), 1, 100, "records"),
    (spread(2047, 32, 70), 1, 128, "records"),         # a block less than wavefronts, as many and one more
    (spread(2048, 32, 70), 1, 128, "records"),
    (spread(2049, 32, 70), 1, 128, "records"),
    (spread(500, 16, 60, 5), 4, 64, "records"),        # 2000 blocks of 64 segments
    (spread(510, 9, 60), 7, 65, "records"),            # 3570 of 63
    ([64 * 16] * 8, 8, 64, "records"),
    ([128 * 16] * 32, 1, 128, "records"),
    ([48 * 16, 5, 0, 700] * 8, 1, 49, "whole on the device"),      # by the bounds they may be longer, but none is
    ([0] * 4, 8, 49, "whole on the device"),                       # nothing at all
    (spread(300, 32, 49), 1, 500, "records"),
    (spread(2047, 64, 900), 1, 1000, "records"),       # one request has much of the wavefronts
    (spread(4096, 32, 3000), 1, 3000, "records"),
    (spread(513, 8, 100, 2), 8, 200, "records"),
    ([48 * 16, 5, 0, 700] * 8, 2, 300, "whole on the device"),
]


def workload(lens, heads, room, **kw):
    return wl.custom(lens, heads, heads, seed=90 + len(lens), num_pool_blocks=sum((n + 15) // 16 for n in lens) + 1, head_dim=64,
                     maxb=room, **kw)


def peaked(k):
    """K so that the records of a segment have unlike maxima."""
    return wl.f32_to_bf16_bits(np.asarray(wl.bf16_bits_to_f64(k), dtype=np.float32) * np.float32(3.0))


def check(w, host, got):
    ref = oracle.paged_decode_attn(*host, w.block_tables, w.context_lens, w.scale)
    c = oracle.compare(got, ref)
    assert c["rel_l2"] <= REL_L2 and c["worst_seq_rel_l2"] <= 2 * REL_L2 and abs_error_within_bar(got, ref), c
    for s in np.flatnonzero(w.context_lens == 0):
        assert not got.reshape(w.q_shape())[s].any()


@pytest.mark.parametrize("i", range(len(BATCHES)))
@pytest.mark.parametrize("partition", [0, 64])
def test_batches(device, i, partition):
    lens, heads, room, route = BATCHES[i]
    w = workload(lens, heads, room, partition_size=partition)
    assert routes.route(w) == route
    q, k, v = wl.make_host_tensors(w, poison_unused=True)
    k = peaked(k) if i % 2 else k
    print(f"{i}: {len(lens)} requests, {heads} heads, {route}", flush=True)
    dev = [to_dev(x) for x in (q, k, v, w.block_tables, w.context_lens)]
    need, guard = pkv.pkv_attn_workspace_bytes(shape_of(w)), 1 << 20
    buf = torch.full((2 * guard + need,), 0xA5, dtype=torch.uint8, device=device)
    first = run_attn_dev(w, *dev, workspace=buf[guard:guard + need])
    torch.cuda.synchronize()
    assert bool((buf[:guard] == 0xA5).all()) and bool((buf[guard + need:] == 0xA5).all())
    check(w, (q, k, v), to_bits(first))
    buf.random_(0, 256)
    assert torch.equal(run_attn_dev(w, *dev, workspace=buf[guard:guard + need]), first)   # whoever ends a segment


@pytest.mark.parametrize("i", [0, 3, 5, 7, 9, 12, 14])
def test_8_bit_pools(device, i):
    lens, heads, room, route = BATCHES[i]
    w = workload(lens, heads, room)
    assert routes.route(w, fp8=True) == route
    q, k8, v8 = wl.make_host_tensors_fp8(w, KS, VS, poison_unused=True)
    print(f"fp8 {i}: {len(lens)} requests, {heads} heads, {route}", flush=True)
    check_fp8(w, q, k8, v8, run_fp8(w, q, k8, v8), f"fp8 {route}")


@pytest.mark.parametrize("room", [64, 800])
def test_replays(device, room):
    """One launch, replayed with lengths that take it from one way to the next: nothing of an earlier replay may be left over."""
    steps = [[60] * 8, [3, 48, 0, 1, 7, 48, 2, 9], [50, 2, 0, 1, 7, 48, 2, 9], [32] * 7 + [51], [49] + [1] * 7]
    if room > 64:
        steps += [[700, 0, 0, 0, 0, 0, 0, 1], [0] * 7 + [160], [90] * 8]
    w = workload([16 * int(b) for b in np.max(steps, axis=0)], 8, room)
    q, k, v = wl.make_host_tensors(w)
    dev = [to_dev(x) for x in (q, k, v, w.block_tables, w.context_lens)]
    shape, lens = shape_of(w), dev[4]
    ws = torch.empty(pkv.pkv_attn_workspace_bytes(shape), dtype=torch.uint8, device=device).random_(0, 256)
    out = torch.empty(w.q_shape(), dtype=torch.int16, device=device)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        pkv.paged_decode_attn(*dev, float(w.scale), out, shape, ws, torch.cuda.current_stream())
    for step in steps + steps[1:]:
        w.context_lens[:] = [max(16 * b - 3 * i, 0) for i, b in enumerate(step)]
        assert routes.route(w) == ("records" if max(step) > 48 else "whole on the device")
        lens.copy_(torch.from_numpy(w.context_lens))
        out.fill_(0x7FC1)
        graph.replay()
        torch.cuda.synchronize()
        print(step, flush=True)
        got = to_bits(out)
        assert np.array_equal(got, to_bits(run_attn_dev(w, *dev))), step
        check(w, (q, k, v), got)


@pytest.mark.parametrize("lens,heads", [
    (spread(1280, 32, 49), 1), (spread(1281, 32, 49), 1), (spread(2048, 40, 60, 3), 1), (spread(4096, 64, 64), 1), (spread(512, 9, 64), 7),
    (spread(512, 8, 64), 8), (spread(4097, 64, 66), 1), (spread(3000, 50, 80), 1), ([48 * 16, 5, 0, 700] * 8, 1),
])
def test_the_bound_does_not_change_a_bit(device, lens, heads):
    """Where partial sums are split follows from the lengths alone, whatever the bounds let the host choose."""
    w = workload(lens, heads, 1200)
    q, k, v = wl.make_host_tensors(w)
    dev = [to_dev(x) for x in (peaked(q), k, v, w.block_tables, w.context_lens)]
    print(f"{len(lens)} requests, {heads} heads", flush=True)
    wide = run_attn_dev(w, *dev)
    for bound in (max(lens), max(lens) + 1, 128 * 16, 5000):
        assert torch.equal(run_attn_dev(w, *dev, max_context_len=bound), wide), bound
