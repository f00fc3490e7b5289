"""K on its way from the pool to the matrix cores at D = 128: turned in LDS where there is room, loaded in operand order
where the records of the query heads leave none (bf16: 16 per KV head, 15 from 640 requests, 14 from 1664; e4m3: 16 from 1664).
Both against the oracle, on shares of zero, one and many blocks, with NaN in the slots behind a request's end."""
import numpy as np
import pytest

import oracle
from paper_2602_11530_amd import workloads as wl

from gpu_util import REL_L2, abs_error_within_bar, run_attn
from test_gpu_fp8kv import KS, VS, check as check_fp8, run_fp8

pytestmark = pytest.mark.gpu

LENS = [1, 17, 0, 16, 333, 2049, 6001]


def heads_and_batch():
    """(query heads per KV head, empty requests behind LENS): the prefix arrays of the batch take LDS too."""
    return [(12, 0), (13, 0), (13, 2000), (14, 0), (14, 2000), (15, 0), (15, 2000), (16, 0), (16, 2000)]


@pytest.mark.parametrize("G,more", heads_and_batch())
@pytest.mark.parametrize("P", [0, 64])
def test_bf16(device, G, more, P):
    w = wl.custom(LENS + [0] * more, G, 1, seed=70 + G, num_pool_blocks=560, partition_size=P)
    q, k, v = wl.make_host_tensors(w, poison_unused=True)
    print(f"G={G} S={w.num_seqs} P={P}", flush=True)
    got = run_attn(w, q, k, v)
    ref = oracle.paged_decode_attn(q, k, v, w.block_tables, w.context_lens, w.scale)
    c = oracle.compare(got, ref)
    assert c["rel_l2"] <= REL_L2 and c["worst_seq_rel_l2"] <= 2 * REL_L2 and abs_error_within_bar(got, ref), c
    assert np.isfinite(wl.bf16_bits_to_f64(got)).all()


@pytest.mark.parametrize("G,more", heads_and_batch())
def test_fp8(device, G, more):
    w = wl.custom(LENS + [0] * more, G, 1, seed=90 + G, num_pool_blocks=560)
    q, k8, v8 = wl.make_host_tensors_fp8(w, KS, VS, poison_unused=True)
    print(f"fp8 G={G} S={w.num_seqs}", flush=True)
    check_fp8(w, q, k8, v8, run_fp8(w, q, k8, v8), f"fp8 G={G}")
