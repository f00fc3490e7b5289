"""D = 128 in bf16 has two launches, by the bounds (short_at_128), which differ in the order of the loads only: they agree bit for bit,
and each with the oracle.  Shares of zero, one, two, some and many blocks, one segment and many, one workgroup to a segment and in
several layers."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_11530_amd import workloads as wl

from gpu_util import REL_L2, abs_error_within_bar, run_attn_dev, shape_of, to_bits, to_dev
from test_gpu_layer_chain import device_layers, layers_call

pytestmark = pytest.mark.gpu

WAVES = 2048


def is_short(w, max_context_len=0):
    blocks = ((max_context_len or w.max_blocks_per_seq * w.block_size) + 15) // 16
    return w.num_seqs * w.num_kv_heads * blocks <= 16 * WAVES


def batch(lens, hq, hkv, P, wide):
    """Its table is as wide as the bounds of a batch with long shares ask for, or just wide enough."""
    blocks = sum((n + 15) // 16 for n in lens)
    width = 16 * WAVES // (len(lens) * hkv) + 1 if wide else 0
    return wl.custom(lens, hq, hkv, seed=79, num_pool_blocks=blocks + 2, partition_size=P, maxb=max(width, max(lens) // 16 + 1))


BATCHES = pytest.mark.parametrize("lens,hq,hkv,P", [
    ([250, 17, 300, 64], 8, 2, 0),                           # a workgroup to a segment
    ([400] + [5, 0, 16, 17] * 20, 8, 8, 0),                  # a block or none
    ([600, 1, 0, 37, 512, 250] * 8, 40, 8, 64),              # two blocks, runs of 4
    ([8191], 40, 8, 0), ([30000], 8, 1, 0), ([9000, 30], 16, 1, 512),   # a few segments; one; no room to turn K
    ([2600 + 7 * i for i in range(18)] + [0], 10, 2, 0)])    # 3
@BATCHES
def test_both_launches(device, lens, hq, hkv, P):
    out = []
    for wide in (True, False):
        w = batch(lens, hq, hkv, P, wide)
        assert is_short(w) != wide
        q, k, v = wl.make_host_tensors(w, poison_unused=True)
        print(f"{len(lens)} requests, {hq}/{hkv} heads, wide {wide}", flush=True)
        out.append(run_attn_dev(w, *[to_dev(x) for x in (q, k, v, w.block_tables, w.context_lens)]))
        torch.cuda.synchronize()
        ref = oracle.paged_decode_attn(q, k, v, w.block_tables, w.context_lens, w.scale)
        c = oracle.compare(to_bits(out[-1]), ref)
        assert c["rel_l2"] <= REL_L2 and c["worst_seq_rel_l2"] <= 2 * REL_L2 and abs_error_within_bar(to_bits(out[-1]), ref), c
        assert np.isfinite(wl.bf16_bits_to_f64(to_bits(out[-1]))).all()
        # the same tensors under the other launch's bounds (the tight one takes the wide table, and the short launch)
        if wide:
            other = run_attn_dev(w, *[to_dev(x) for x in (q, k, v, w.block_tables, w.context_lens)], max_context_len=max(lens))
            assert is_short(w, max(lens)) and torch.equal(out[-1], other)


@pytest.mark.parametrize("lens", [[600, 1, 0, 37, 512, 250] * 4, [30, 100, 90]])
def test_layers(device, lens):
    w = batch(lens, 16, 8, 0, True)
    assert not is_short(w) and is_short(w, max(lens))
    dev = device_layers(w, 3, 9)
    t_d, l_d = to_dev(w.block_tables), to_dev(w.context_lens)
    single = [run_attn_dev(w, q, k, v, t_d, l_d) for q, k, v in dev]
    for shape in (shape_of(w), shape_of(w, max_context_len=max(lens))):
        assert all(torch.equal(a, b) for a, b in zip(layers_call(w, dev, t_d, l_d, shape), single))
