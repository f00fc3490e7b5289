"""D = 256 has two launches, by the bounds (large_at_256), which differ in the order of the loads (bf16) or in the way of K to the
matrix cores (e4m3) only: they agree bit for bit, and each with the oracle.  Shares of zero, one, two, some and many blocks, one segment and many, and in
several layers."""
import copy

import numpy as np
import pytest
import torch

import oracle
from paper_2602_11530_amd import workloads as wl

from gpu_util import REL_L2, abs_error_within_bar, run_attn_dev, shape_of, to_bits, to_dev
from test_gpu_fp8kv import KS, VS, check as check_fp8, run_fp8
from test_gpu_layer_chain import device_layers, layers_call

pytestmark = pytest.mark.gpu

WAVES = 1024


def is_large(w, max_context_len=0):
    blocks = ((max_context_len or w.max_blocks_per_seq * w.block_size) + 15) // 16
    return w.num_seqs * w.num_kv_heads * blocks >= 24 * WAVES


BATCHES = pytest.mark.parametrize("lens,hq,hkv,P", [
    ([400] + [5, 0, 16, 17] * 20, 8, 8, 0),               # most wavefronts have a block, some none
    ([600, 1, 0, 37, 512, 250] * 4, 16, 8, 64),           # shares of 4 and 5, runs of 4
    ([9000], 8, 1, 0), ([7000, 30], 40, 8, 0),            # one segment; a few
    ([2600 + 7 * i for i in range(20)] + [0], 8, 8, 512)])   # 26, large by the tight bound too
def batch(lens, hq, hkv, P):
    """Its table is wide enough for the bounds of a large batch."""
    blocks = sum((n + 15) // 16 for n in lens)
    return wl.custom(lens, hq, hkv, seed=77, num_pool_blocks=blocks + 2, head_dim=256, partition_size=P,
                     maxb=24 * WAVES // (len(lens) * hkv) + max(lens) // 16 + 1)


@BATCHES
def test_bf16(device, lens, hq, hkv, P):
    w, tight = batch(lens, hq, hkv, P), max(lens)
    assert is_large(w) and (not is_large(w, tight) or tight > 2000)
    q, k, v = wl.make_host_tensors(w, poison_unused=True)
    dev = [to_dev(x) for x in (q, k, v, w.block_tables, w.context_lens)]
    print(f"{len(lens)} requests, {hq}/{hkv} heads", flush=True)
    large = run_attn_dev(w, *dev)
    small = run_attn_dev(w, *dev, max_context_len=tight)
    torch.cuda.synchronize()
    assert torch.equal(large, small)
    ref = oracle.paged_decode_attn(q, k, v, w.block_tables, w.context_lens, w.scale)
    c = oracle.compare(to_bits(large), ref)
    assert c["rel_l2"] <= REL_L2 and c["worst_seq_rel_l2"] <= 2 * REL_L2 and abs_error_within_bar(to_bits(large), ref), c
    assert np.isfinite(wl.bf16_bits_to_f64(to_bits(large))).all()


@BATCHES
def test_fp8(device, lens, hq, hkv, P):
    w = batch(lens, hq, hkv, P)
    narrow = copy.copy(w)
    narrow.block_tables = np.ascontiguousarray(w.block_tables[:, :(max(lens) + 15) // 16])
    assert is_large(w) and (not is_large(narrow) or max(lens) > 2000)
    q, k8, v8 = wl.make_host_tensors_fp8(w, KS, VS, poison_unused=True)
    print(f"fp8 {len(lens)} requests, {hq}/{hkv} heads", flush=True)
    large = run_fp8(w, q, k8, v8)
    assert np.array_equal(large, run_fp8(narrow, q, k8, v8))
    check_fp8(w, q, k8, v8, large, "fp8 large")


def test_layers(device):
    lens = [600, 1, 0, 37, 512, 250] * 4
    w = wl.custom(lens, 16, 8, seed=78, num_pool_blocks=1400, head_dim=256, maxb=150)
    assert is_large(w) and not is_large(w, 600)
    dev = device_layers(w, 3, 9)
    t_d, l_d = to_dev(w.block_tables), to_dev(w.context_lens)
    single = [run_attn_dev(w, q, k, v, t_d, l_d) for q, k, v in dev]
    for shape in (shape_of(w), shape_of(w, max_context_len=600)):
        assert all(torch.equal(a, b) for a, b in zip(layers_call(w, dev, t_d, l_d, shape), single))
