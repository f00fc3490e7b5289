"""GPU tests of how the partial results of a segment (request, KV head) meet: inside a wavefront's share, in a
workgroup, over several workgroups (a record for each), in batches cut along their segments; on workspaces whose earlier
contents vary, called repeatedly and replayed from a graph."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import MAX_ABS, REL_L2, abs_error_within_bar, device_tensors, run_attn_dev, shape_of, to_bits, to_dev
from paper_2602_11530_amd import binding as pkv
from paper_2602_11530_amd import workloads as wl

pytestmark = pytest.mark.gpu

# lengths, query heads, KV heads, head dim
SHAPES = [
    ([33000], 8, 1, 128),            # one segment: a record of every workgroup
    ([17000, 16000], 8, 2, 64),      # a boundary inside a workgroup
    ([9000, 1, 20000], 5, 1, 256),   # two long segments and a one-block one between them
    ([4200] * 8, 16, 1, 128),        # 32 records each
    ([4300] * 7 + [2000], 16, 1, 128),
    ([2048] * 64, 8, 4, 128),        # many; shares and segments end together: nothing is shared
    ([1, 16, 17, 0, 33] * 60, 10, 2, 64),    # many segments inside one share
    ([16] * 700 + [30000], 12, 1, 128),      # staged rows fill up; then one long segment, in one set of threads
    ([16] * 100 + [30000], 2, 1, 64),        # many, one of them over nearly all workgroups: 16 sets of threads, several
    ([16] * 100 + [30000], 5, 1, 64),        # reads for each; sets that do not fill the workgroup
    ([16] * 100 + [30000], 4, 1, 256),
    ([16] * 70 + [9000, 0, 7000], 8, 1, 256),
    ([5000, 900, 1, 3000] * 18, 5, 1, 256),  # many, shared by two or three workgroups each
    ([700, 0, 5000, 3, 129], 40, 8, 128),
    ([384, 0, 1, 130, 17], 8, 2, 128),       # cut along the segments: the longest that is (3 blocks per wavefront)
    ([385, 0, 1, 130, 17], 8, 2, 128),       # and one token beyond
    ([768, 0, 1, 130, 17], 8, 2, 128),
    ([192, 16, 15, 0], 8, 1, 256),
    ([193, 16, 15, 0], 8, 1, 256),
    ([768, 0, 1, 130, 17], 8, 2, 64),        # 4 KiB blocks: 6 per wavefront
    ([769, 0, 1, 130, 17], 8, 2, 64),
    ([768, 5, 300, 0] * 5, 40, 8, 128),      # more than 64 segments: 6 per wavefront
    ([769, 5, 300, 0] * 5, 40, 8, 128),
    ([384, 16, 15, 0] * 8, 16, 8, 256),
    ([768, 5, 300, 0] * 8, 32, 8, 64),       # as many segments as workgroups
    ([768, 5, 300, 0] * 8 + [64], 32, 8, 64),
    ([2000, 30] * 4, 8, 8, 64),              # records of one head
    ([2000, 30] * 4, 7, 7, 64),
    ([16 * 2047], 8, 1, 64),                 # a block less than wavefronts, as many and one more
    ([16 * 2048 - 5], 8, 1, 128),
    ([16 * 2049], 8, 1, 128),
    ([16 * 1023, 0], 8, 1, 256),
    ([16 * 1024, 16], 8, 1, 256),
    ([16 * 255, 3, 0, 160], 16, 1, 128),     # fewer wavefronts than twice the workgroups, and an empty request
    ([16 * 80] * 2, 8, 8, 128),              # 16 segments, ten records each, and eleven of some
    ([16 * 80, 16 * 81], 8, 8, 128),
    ([16 * 128, 0, 16 * 32], 16, 4, 256),
    ([16 * 128, 0, 16 * 33], 16, 4, 256),
    ([16 * 1000, 40] * 4, 64, 4, 128),       # 32 segments
    ([16 * 200] * 8 + [9], 14, 7, 64),       # 63
    ([16 * 200] * 8 + [9], 56, 7, 64),
    ([9000, 5, 7000, 400, 1], 5, 1, 64),     # a few long segments, items that do not divide the workgroup
    ([9000, 5, 7000, 400, 1], 4, 1, 256),    # two threads for each 16 bytes, and one
    ([9000, 5, 7000, 400, 1], 8, 1, 256),
    ([3000, 0, 5000] * 3, 9, 9, 64),         # records of one head
]


def setup(lens, hq, hkv, dim, seed):
    w = wl.custom(lens, hq, hkv, head_dim=dim, seed=seed)
    q, k, v = device_tensors(w)
    return w, (q.view(torch.int16), k.view(torch.int16), v.view(torch.int16), to_dev(w.block_tables), to_dev(w.context_lens))


def reference(w, dev):
    host = [to_bits(t).reshape(s) for t, s in zip(dev[:3], (w.q_shape(), w.pool_shape(), w.pool_shape()))]
    return oracle.paged_decode_attn(*host, w.block_tables, w.context_lens, w.scale)


@pytest.mark.parametrize("i", range(len(SHAPES)))
@pytest.mark.parametrize("partition", [0, 64])
def test_shared_segments(device, i, partition):
    w, dev = setup(*SHAPES[i], seed=300 + i)
    shape = shape_of(w, partition)
    ws = torch.full((pkv.pkv_attn_workspace_bytes(shape),), 0xFF, dtype=torch.uint8, device=device)
    first = to_bits(run_attn_dev(w, *dev, partition_size=partition, workspace=ws))
    ref = reference(w, dev)
    c = oracle.compare(first, ref)
    assert abs_error_within_bar(first, ref) and c["rel_l2"] <= REL_L2, c
    for fill in (None, 0, "noise"):
        if fill == 0:
            ws.zero_()
        elif fill:
            ws.random_(0, 256)
        again = to_bits(run_attn_dev(w, *dev, partition_size=partition, workspace=ws))
        assert np.array_equal(first, again)   # whoever finishes a segment, its rows are the same bits


@pytest.mark.parametrize("hq,hkv", [(8, 1), (16, 2), (34, 17)])
def test_replays_with_growing_lengths(device, hq, hkv):
    """What becomes of a batch is decided on the device: replays of one launch are cut along the segments or leave
    workgroups' records, and nothing of an earlier one may be left over."""
    w, (q, k, v, tables, lens) = setup([40, 3000, 9, 12000], hq, hkv, 128, seed=400)
    w.context_lens[:] = [17, 16, 9, 33]
    lens.copy_(torch.from_numpy(w.context_lens))
    shape = shape_of(w)
    ws = torch.empty(pkv.pkv_attn_workspace_bytes(shape), dtype=torch.uint8, device=device)
    out = torch.empty(w.q_shape(), dtype=torch.int16, device=device)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        pkv.paged_decode_attn(q, k, v, tables, lens, float(w.scale), out, shape, ws, torch.cuda.current_stream())
    for step in ([17, 16, 9, 33], [40, 3000, 9, 12000], [1, 2900, 0, 12000], [40, 0, 0, 700], [40, 3000, 9, 11999]):
        w.context_lens[:] = step
        lens.copy_(torch.from_numpy(w.context_lens))
        out.fill_(0x7FC1)
        graph.replay()
        torch.cuda.synchronize()
        got = to_bits(out)
        eager = to_bits(run_attn_dev(w, q, k, v, tables, lens))
        assert np.array_equal(got, eager), step
        ref = reference(w, (q, k, v))
        c = oracle.compare(got, ref)
        assert c["max_abs"] <= MAX_ABS and c["rel_l2"] <= REL_L2, (step, c)


@pytest.mark.parametrize("lens,hq,hkv,dim", [
    ([700, 0, 5000, 3, 129, 16, 2000, 31, 1], 40, 8, 128),   # several layers to a launch
    ([3000] * 40, 16, 2, 64),
    ([700, 5000, 129], 16, 8, 256),                          # few segments, likewise
    ([900, 0, 30, 17] * 8, 1, 1, 64),                        # the shortest records
    ([40, 3, 768, 0], 8, 2, 128),                            # cut along the segments
])
@pytest.mark.parametrize("layers", [1, 3, 9])
def test_layers_in_shared_launches(device, lens, hq, hkv, dim, layers):
    """The layers call gives the single calls' bits, also where one layer's output is the next one's q."""
    w, (q, k, v, tables, lens_d) = setup(lens, hq, hkv, dim, seed=500 + layers)
    shape = shape_of(w)
    ws = torch.empty(pkv.pkv_attn_workspace_bytes(shape), dtype=torch.uint8, device=device)
    qs = [torch.roll(q, i, 0).contiguous() for i in range(layers)]
    ks = [torch.roll(k, i, 0).contiguous() for i in range(layers)]
    vs = [torch.roll(v, 2 * i, 0).contiguous() for i in range(layers)]
    for chained in (False, True):
        outs = [torch.full_like(q, 0x7FC1) for _ in range(layers)]
        want = []
        for i in range(layers):
            src = want[i - 1] if chained and i % 2 else qs[i]
            want.append(run_attn_dev(w, src, ks[i], vs[i], tables, lens_d))
        inputs = [outs[i - 1] if chained and i % 2 else qs[i] for i in range(layers)]
        pkv.paged_decode_attn_layers(inputs, ks, vs, tables, lens_d, float(w.scale), outs, shape, ws)
        torch.cuda.synchronize()
        for i in range(layers):
            assert torch.equal(outs[i], want[i]), (chained, i)


@pytest.mark.parametrize("lens,hq,hkv,dim,bound", [
    ([40, 3, 768, 0] * 4, 40, 8, 128, 768),       # 128 segments, cut along them in one launch: nothing left for a reduce pass
    ([40, 3, 384, 0] * 8, 16, 8, 256, 384),       # as many segments as workgroups
    ([16] * 13, 10, 5, 64, 16),                   # a block each
    ([40, 3, 769, 0] * 4, 40, 8, 128, 769),       # a token beyond: records, four layers to a launch at most
])
@pytest.mark.parametrize("layers", [5, 8, 9])
def test_layers_stay_inside_the_workspace(device, lens, hq, hkv, dim, bound, layers):
    w, (q, k, v, tables, lens_d) = setup(lens, hq, hkv, dim, seed=600 + layers)
    shape = shape_of(w, max_context_len=bound)
    need, guard = pkv.pkv_attn_workspace_bytes(shape), 8 << 20   # more than any layer's room
    buf = torch.full((2 * guard + need,), 0xA5, dtype=torch.uint8, device=device)
    qs = [torch.roll(q, i, 0).contiguous() for i in range(layers)]
    ks = [torch.roll(k, i, 0).contiguous() for i in range(layers)]
    vs = [torch.roll(v, 2 * i, 0).contiguous() for i in range(layers)]
    outs = [torch.full_like(q, 0x7FC1) for _ in range(layers)]
    pkv.paged_decode_attn_layers(qs, ks, vs, tables, lens_d, float(w.scale), outs, shape, buf[guard:guard + need])
    torch.cuda.synchronize()
    assert bool((buf[:guard] == 0xA5).all()) and bool((buf[guard + need:] == 0xA5).all())
    for i in range(layers):
        want = run_attn_dev(w, qs[i], ks[i], vs[i], tables, lens_d, max_context_len=bound)
        assert torch.equal(outs[i], want), i


@pytest.mark.parametrize("lens,hq,hkv,dim", [
    ([700, 0, 5000, 3, 129, 16, 2000, 31, 1], 40, 8, 128),   # more than 64 segments
    ([3000, 40, 0, 700], 16, 8, 128),                        # few
    ([1500, 0, 30] * 12, 4, 1, 64),
    ([900, 0, 30, 17] * 8, 1, 1, 64),                        # the shortest records
    ([9000, 300], 8, 1, 128),
    ([40, 3, 300, 0], 8, 2, 128),                            # cut along the segments
])
def test_output_over_inputs(device, lens, hq, hkv, dim):
    """The inputs are read as they were before the call, also where the output lies over q or over a pool."""
    w, (q, k, v, tables, lens_d) = setup(lens, hq, hkv, dim, seed=700)
    want = run_attn_dev(w, q, k, v, tables, lens_d)
    ref = oracle.paged_decode_attn(*[to_bits(t).reshape(s) for t, s in zip((q, k, v), (w.q_shape(), w.pool_shape(), w.pool_shape()))],
                                   w.block_tables, w.context_lens, w.scale)
    shape = shape_of(w)
    ws = torch.empty(pkv.pkv_attn_workspace_bytes(shape), dtype=torch.uint8, device=device)

    def check(out, what, exact):
        torch.cuda.synchronize()
        if exact:
            assert torch.equal(out, want), what
        c = oracle.compare(to_bits(out), ref)
        assert abs_error_within_bar(to_bits(out), ref) and c["rel_l2"] <= REL_L2, (what, c)

    n = q.numel()
    for shift in (0, 8, dim, -dim, hq * dim, -3 * hq * dim):   # elements
        buf = torch.zeros(n + 2 * abs(shift), dtype=torch.int16, device=device)
        at = abs(shift)
        buf[at:at + n] = q.reshape(-1)
        out = buf[at + shift:at + shift + n].view(q.shape)
        run_attn_dev(w, buf[at:at + n].view(q.shape), k, v, tables, lens_d, workspace=ws, out=out)
        check(out, shift, shift == 0)
    pool = k.clone()
    flat = pool.view(-1)
    out = flat[flat.numel() - n:].view(q.shape)
    run_attn_dev(w, q, pool, v, tables, lens_d, workspace=ws, out=out)
    check(out, "K pool", False)
    # in the layers call the next layer reads what this one wrote
    pool = k.clone()
    flat = pool.view(-1)
    outs = [flat[flat.numel() - n:].view(q.shape), torch.empty_like(q)]
    pkv.paged_decode_attn_layers([q, q], [pool, pool], [v, v], tables, lens_d, float(w.scale), outs, shape, ws)
    check(outs[0], "first layer", False)
    assert torch.equal(outs[1], run_attn_dev(w, q, pool, v, tables, lens_d))
