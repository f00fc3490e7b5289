"""bf16 at D = 256 has two launches, by the bounds (late_at_256): V is asked for a block ahead, or when K is there.  Only the order
of the loads differs, so they agree bit for bit; and each with the oracle.  Shares of zero, one, two, some and many blocks, by
rows, by workgroups and in several layers."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_11530_amd import workloads as wl

from gpu_util import REL_L2, abs_error_within_bar, run_attn_dev, shape_of, to_bits, to_dev
from test_gpu_layer_chain import device_layers, layers_call

pytestmark = pytest.mark.gpu

WAVES = 1024


def is_late(w, max_context_len=0):
    blocks = ((max_context_len or w.max_blocks_per_seq * w.block_size) + 15) // 16
    return w.num_seqs * w.num_kv_heads * blocks >= 24 * WAVES


@pytest.mark.parametrize("lens,hq,hkv,P", [
    ([400] + [5, 0, 16, 17] * 20, 8, 8, 0),               # most wavefronts have a block, some none
    ([600, 1, 0, 37, 512, 250] * 4, 16, 8, 64),           # shares of 4 and 5, runs of 4
    ([9000], 8, 1, 0), ([7000, 30], 40, 8, 0),            # by rows; a few segments
    ([2600 + 7 * i for i in range(20)] + [0], 8, 8, 512)])   # 26, which is late by the tight bound too
def test_both_orders_agree(device, lens, hq, hkv, P):
    blocks = sum((n + 15) // 16 for n in lens)
    w = wl.custom(lens, hq, hkv, seed=77, num_pool_blocks=blocks + 2, head_dim=256, partition_size=P,
                  maxb=24 * WAVES // (len(lens) * hkv) + max(lens) // 16 + 1)
    tight = max(lens)
    assert is_late(w) and (not is_late(w, tight) or blocks * hkv > 24 * WAVES)
    q, k, v = wl.make_host_tensors(w, poison_unused=True)
    dev = [to_dev(x) for x in (q, k, v, w.block_tables, w.context_lens)]
    print(f"{len(lens)} requests, {hq}/{hkv} heads", flush=True)
    late = run_attn_dev(w, *dev)
    early = run_attn_dev(w, *dev, max_context_len=tight)
    torch.cuda.synchronize()
    assert torch.equal(late, early)
    ref = oracle.paged_decode_attn(q, k, v, w.block_tables, w.context_lens, w.scale)
    c = oracle.compare(to_bits(late), ref)
    assert c["rel_l2"] <= REL_L2 and c["worst_seq_rel_l2"] <= 2 * REL_L2 and abs_error_within_bar(to_bits(late), ref), c
    assert np.isfinite(wl.bf16_bits_to_f64(to_bits(late))).all()


def test_layers_in_both_orders(device):
    lens = [600, 1, 0, 37, 512, 250] * 4
    w = wl.custom(lens, 16, 8, seed=78, num_pool_blocks=1400, head_dim=256, maxb=150)
    assert is_late(w) and not is_late(w, 600)
    dev = device_layers(w, 3, 9)
    t_d, l_d = to_dev(w.block_tables), to_dev(w.context_lens)
    single = [run_attn_dev(w, q, k, v, t_d, l_d) for q, k, v in dev]
    for shape in (shape_of(w), shape_of(w, max_context_len=600)):
        assert all(torch.equal(a, b) for a, b in zip(layers_call(w, dev, t_d, l_d, shape), single))
