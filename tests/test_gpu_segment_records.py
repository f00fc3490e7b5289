"""GPU parity of the reduce pass over workgroups' records by how many of them a segment has: up to a turn of loads (4), two turns' worth (8), one
more, from where a segment has several workgroups and several sets of lanes in each, hundreds; few segments and many; the smallest
and the largest rows.  Peaked scores, so that the records of a segment have unlike maxima, in one of them by far the largest."""
import numpy as np
import pytest
import torch

import oracle
import routes
from paper_2602_11530_amd import workloads as wl

from gpu_util import REL_L2, abs_error_within_bar, run_attn_dev, to_bits, to_dev

pytestmark = pytest.mark.gpu


# lengths, and how many records their segments have, among others, at one KV head and at two
LENGTHS = [
    ([900 + 3 * i for i in range(70)], {4, 5}, {2, 3}),
    ([2600, 40] * 36 + [0, 7], {1, 2, 7, 8}, {1, 2, 4, 5}),
    ([1300 + 24 * i for i in range(31)], {7, 8, 9, 10, 11}, {4, 5, 6}),
    ([2100 + 51 * i for i in range(17)], {13, 15, 16, 17, 18}, {7, 8, 9, 10}),
    ([4200 + 100 * i for i in range(8)], {30, 31, 32, 33, 34, 35}, {15, 16, 17, 18}),
    ([3000] * 6, set(), {22}),
    ([12000] + [1] * 70, {1}, {1, 94, 95}),
]


@pytest.mark.parametrize("hq,hkv,dim", [(5, 1, 128), (1, 1, 64), (16, 1, 64), (16, 1, 128), (1, 1, 256), (8, 1, 256), (10, 2, 128)])
@pytest.mark.parametrize("i", range(len(LENGTHS)))
def test_records_of_a_segment(device, hq, hkv, dim, i):
    lens, *counts = LENGTHS[i]
    w = wl.custom(lens, hq, hkv, seed=83 + dim, head_dim=dim)
    assert routes.route(w) == "records" and counts[hkv - 1] <= set(routes.records(w))
    q, k, v = wl.make_host_tensors(w, poison_unused=True)
    k = wl.f32_to_bf16_bits(np.asarray(wl.bf16_bits_to_f64(k), dtype=np.float32) * np.float32(3.0))
    print(f"{len(lens)} requests, {hq}/{hkv} heads, D {dim}", flush=True)
    out = run_attn_dev(w, *[to_dev(x) for x in (q, k, v, w.block_tables, w.context_lens)])
    torch.cuda.synchronize()
    ref = oracle.paged_decode_attn(q, k, v, w.block_tables, w.context_lens, w.scale)
    c = oracle.compare(to_bits(out), ref)
    assert c["rel_l2"] <= REL_L2 and c["worst_seq_rel_l2"] <= 2 * REL_L2 and abs_error_within_bar(to_bits(out), ref), c
