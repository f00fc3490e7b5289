"""GPU parity of the reduce pass over workgroups' records by how many of them a segment has: up to a turn of loads, two turns' worth, one more, enough
for several workgroups to a segment and for several sets of lanes in each, hundreds; few segments and many; the smallest and the
largest rows.  Peaked scores, so that the records of a segment have unlike maxima, in one of them by far the largest."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_11530_amd import workloads as wl

from gpu_util import REL_L2, abs_error_within_bar, run_attn_dev, to_bits, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,dim", [(5, 1, 128), (1, 1, 64), (16, 1, 64), (16, 1, 128), (1, 1, 256), (8, 1, 256), (10, 2, 128)])
@pytest.mark.parametrize("lens", [
    [3000] * 6,                       # tens of records to a segment, few segments
    [900 + 3 * i for i in range(40)],   # half a dozen
    [1150] * 32,                      # eight and nine
    [12000] + [1] * 70,               # hundreds and none, many segments
    [2600, 40] * 36 + [0, 7],         # two to five
])
def test_records_of_a_segment(device, hq, hkv, dim, lens):
    w = wl.custom(lens, hq, hkv, seed=83 + dim, head_dim=dim)
    q, k, v = wl.make_host_tensors(w, poison_unused=True)
    k = wl.f32_to_bf16_bits(np.asarray(wl.bf16_bits_to_f64(k), dtype=np.float32) * np.float32(3.0)) if hq == 5 else k
    print(f"{len(lens)} requests, {hq}/{hkv} heads, D {dim}", flush=True)
    out = run_attn_dev(w, *[to_dev(x) for x in (q, k, v, w.block_tables, w.context_lens)])
    torch.cuda.synchronize()
    ref = oracle.paged_decode_attn(q, k, v, w.block_tables, w.context_lens, w.scale)
    c = oracle.compare(to_bits(out), ref)
    assert c["rel_l2"] <= REL_L2 and c["worst_seq_rel_l2"] <= 2 * REL_L2 and abs_error_within_bar(to_bits(out), ref), c
