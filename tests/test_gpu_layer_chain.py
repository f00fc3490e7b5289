"""Several layers to a launch: a workgroup goes from its range of one layer to the same range of the next with that layer's first
loads under way.  Bit for bit what single calls give, on shares that end inside, at and behind a window of 64 block
descriptors, on batches with fewer blocks than wavefronts, and with the same count of refused ids."""
import numpy as np
import pytest
import torch

from paper_2602_11530_amd import binding as pkv
from paper_2602_11530_amd import workloads as wl

import routes
from gpu_util import run_attn_dev, shape_of, to_dev

pytestmark = pytest.mark.gpu


def layers_call(w, dev, t_d, l_d, shape):
    ws = torch.empty(pkv.pkv_attn_workspace_bytes(shape), dtype=torch.uint8, device="cuda:0").fill_(0xA5)
    outs = [torch.full(w.q_shape(), 0x7FC1, dtype=torch.int16, device="cuda:0") for _ in dev]
    pkv.paged_decode_attn_layers([d[0] for d in dev], [d[1] for d in dev], [d[2] for d in dev], t_d, l_d, float(w.scale), outs,
                                 shape, ws)
    torch.cuda.synchronize()
    return outs


def chained(w):
    """Do workgroups go from layer to layer?  Not where each segment has one by the bounds."""
    return routes.route(w) != "whole"


def device_layers(w, n, seed):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)

    def normal(shape):
        return torch.randn(shape, generator=g, device="cuda:0").to(torch.bfloat16).view(torch.int16)

    return [(normal(w.q_shape()), normal(w.pool_shape()), normal(w.pool_shape())) for _ in range(n)]


# blocks per share at 2048 wavefronts (1024 at D = 256): the first two have a workgroup for each segment, the layers side by
# side; then 51, 69, 63, 64, 129, 64 and, of a few segments, 2 and 66
@pytest.mark.parametrize("dim,lens,hq,hkv", [
    (128, [40, 0, 17] * 24, 2, 2), (128, [300] * 70 + [0] * 5, 4, 2), (64, [5000 + 13 * i for i in range(40)], 8, 8),
    (128, [15700, 15800, 15900] * 6 + [0], 8, 8), (128, [16120] * 16 + [1] * 4, 8, 8), (128, [16384 + 40] * 16, 8, 8),
    (128, [33000] * 16, 8, 8), (256, [8200] * 16 + [17] * 3, 8, 8), (64, [8000, 0, 31], 40, 8), (256, [17000] * 8, 8, 8)])
def test_equals_single_calls(device, dim, lens, hq, hkv):
    blocks = sum((n + 15) // 16 for n in lens) + 3
    w = wl.custom(lens, hq, hkv, seed=61, num_pool_blocks=blocks, head_dim=dim)
    assert chained(w) == (max(lens) > 1000)
    dev = device_layers(w, 5, 7)
    t_d, l_d = to_dev(w.block_tables), to_dev(w.context_lens)
    print(f"D={dim} S={len(lens)} {hq}/{hkv} blocks={blocks}", flush=True)
    single = [run_attn_dev(w, q, k, v, t_d, l_d) for q, k, v in dev]
    for got, want in zip(layers_call(w, dev, t_d, l_d, shape_of(w)), single):
        assert torch.equal(got, want)


# Short shares on the chained path, by a table wider than what is in use: less than a block for each wavefront; no segment
# longer than a workgroup takes (cut along them on the device, some workgroups without any); 3; then exactly 62 to 66, where a
# window of 64 ends before, with and behind the share
@pytest.mark.parametrize("dim,lens,hq,hkv,P", [
    (128, [900] + [40, 0, 17] * 24, 2, 2, 0), (128, [40, 0, 17] * 24, 2, 2, 0), (256, [100, 0, 17] * 24, 8, 2, 0),
    (128, [180, 0] * 70, 16, 8, 64), (64, [180] * 70, 8, 8, 512)] +
    [(64, [256 * k] * 16, 8, 8, 64 if k == 64 else 0) for k in range(62, 67)])
def test_short_shares_equal_single_calls(device, dim, lens, hq, hkv, P):
    blocks = sum((n + 15) // 16 for n in lens) + 3
    w = wl.custom(lens, hq, hkv, seed=63, num_pool_blocks=blocks, head_dim=dim, partition_size=P, maxb=max(60, max(lens) // 16 + 1))
    assert chained(w)
    dev = device_layers(w, 3, 11)
    t_d, l_d = to_dev(w.block_tables), to_dev(w.context_lens)
    print(f"D={dim} S={len(lens)} {hq}/{hkv} blocks={blocks} P={P}", flush=True)
    single = [run_attn_dev(w, q, k, v, t_d, l_d) for q, k, v in dev]
    for got, want in zip(layers_call(w, dev, t_d, l_d, shape_of(w)), single):
        assert torch.equal(got, want)


@pytest.mark.expects_id_faults
@pytest.mark.parametrize("n_tokens", [900, 17000])
def test_refused_ids_are_counted_in_every_layer(device, id_faults, n_tokens):
    """Shares of one descriptor window, and of more."""
    lens = [n_tokens] * 16
    w = wl.custom(lens, 8, 8, seed=62, num_pool_blocks=sum((n + 15) // 16 for n in lens))
    dev = device_layers(w, 3, 8)
    tables = w.block_tables.copy()
    tables[3, 5], tables[9, 0], tables[15, -1] = -7, 1 << 30, w.num_pool_blocks
    t_d, l_d = to_dev(tables), to_dev(w.context_lens)
    single = [run_attn_dev(w, q, k, v, t_d, l_d) for q, k, v in dev]
    torch.cuda.synchronize()
    counted = int(id_faults.item())
    assert counted == 3 * 3 * 8      # ids, layers, KV heads
    outs = layers_call(w, dev, t_d, l_d, shape_of(w))
    assert int(id_faults.item()) == 2 * counted
    assert all(torch.equal(a, b) for a, b in zip(outs, single))
