"""Batches whose bounds say that each segment has a workgroup take a launch of their own: it agrees bit for bit with the one that finds out on
the device (the same tensors under wide bounds), and with the oracle.  Lengths around blocks and wavefronts, empty requests, runs of
few tokens, physical blocks of 16, 32 and 64 tokens, refused ids, tables narrower than a wavefront."""
import copy

import numpy as np
import pytest
import torch

import oracle
from paper_2602_11530_amd import workloads as wl

from gpu_util import REL_L2, abs_error_within_bar, run_attn_dev, to_bits, to_dev
from test_gpu_fp8kv import KS, VS, check as check_fp8, run_fp8

pytestmark = pytest.mark.gpu


def longest(D, segments, fp8):   # what the rule allows, in tokens
    waves = 4 if D == 256 else 8
    return 16 * waves * (3 if segments <= 64 and D * (1 if fp8 else 2) >= 256 else 6)


def batches(D, fp8):
    most = longest(D, 8, fp8)
    return [([1], 8, 8, 16, 0), ([0, 16, 17, 0], 8, 2, 16, 0), ([most, most - 1, 15, 130, 128, 127], 8, 1, 32, 64), ([most, 65], 16, 2, 64, 64),
            ([0, 5, 31, 32, 33, 100, 111, 113, 128, 129] * 5, 10 if D != 256 else 8, 2, 16, 16)]


@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("case", range(5))
@pytest.mark.parametrize("fp8", [False, True])
def test_against_the_general_launch(device, D, case, fp8):
    lens, hq, hkv, B, P = batches(D, fp8)[case]
    segments = len(lens) * hkv
    assert segments <= 256 and max(lens) <= longest(D, segments, fp8)
    blocks = sum((n + B - 1) // B for n in lens)
    w = wl.custom(lens, hq, hkv, seed=80 + case, num_pool_blocks=blocks + 2, head_dim=D, block_size=B, partition_size=P,
                  maxb=longest(D, segments, fp8) // B + 1)
    tight = copy.copy(w)
    tight.block_tables = np.ascontiguousarray(w.block_tables[:, :max(1, (max(lens) + B - 1) // B)])
    assert w.max_blocks_per_seq * B > longest(D, segments, fp8)
    print(f"D={D} fp8={fp8} {lens} {hq}/{hkv} B={B}", flush=True)
    if fp8:
        q, k, v = wl.make_host_tensors_fp8(w, KS, VS, poison_unused=True)
        general, whole = run_fp8(w, q, k, v), run_fp8(tight, q, k, v)
        check_fp8(w, q, k, v, whole, "whole")
        assert np.array_equal(general, whole)
        return
    q, k, v = wl.make_host_tensors(w, poison_unused=True)
    general, whole = (to_bits(run_attn_dev(x, *[to_dev(t) for t in (q, k, v, x.block_tables, x.context_lens)])) for x in (w, tight))
    ref = oracle.paged_decode_attn(q, k, v, w.block_tables, w.context_lens, w.scale)
    c = oracle.compare(whole, ref)
    assert c["rel_l2"] <= REL_L2 and c["worst_seq_rel_l2"] <= 2 * REL_L2 and abs_error_within_bar(whole, ref), c
    assert np.array_equal(general, whole)


@pytest.mark.expects_id_faults
@pytest.mark.parametrize("D", [64, 128, 256])
def test_refused_ids(device, id_faults, D):
    lens, B = [100, 40, 0, 17], 32
    w = wl.custom(lens, 8, 2, seed=90, num_pool_blocks=9, head_dim=D, block_size=B, maxb=4)
    q, k, v = wl.make_host_tensors(w)
    dev = [to_dev(t) for t in (q, k, v)]
    wide = copy.copy(w)
    wide.block_tables = np.full((4, 40), -1, np.int32)
    wide.block_tables[:, :4] = w.block_tables
    outs, counts = [], []
    for x in (w, wide):
        tables = x.block_tables.copy()
        tables[0, 1], tables[1, 0], tables[1, 1], tables[3, 0] = 9, -1, 1 << 30, -(1 << 31)
        before = int(id_faults.item())
        outs.append(run_attn_dev(x, *dev, to_dev(tables), to_dev(x.context_lens), check_tables=False))
        torch.cuda.synchronize()
        counts.append(int(id_faults.item()) - before)
    # 2 KV heads times 16-token units: two of request 0's, all three of request 1's, both of request 3's
    assert counts == [14, 14]
    assert torch.equal(*outs)
    assert not outs[0][1].any() and not outs[0][2].any() and not outs[0][3].any() and outs[0][0].any()
