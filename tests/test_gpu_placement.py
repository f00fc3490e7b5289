"""Where a wavefront's blocks lie is found from its first and last position: batches around 64 requests and at the largest number, with runs of
empty requests, windows that reach over one request or over dozens, and head counts that divide nothing, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2602_11530_amd import workloads as wl

from gpu_util import REL_L2, abs_error_within_bar, run_attn

pytestmark = pytest.mark.gpu


def lengths(S, longest, empty, seed):
    rng = np.random.default_rng(seed)
    n = rng.integers(1, longest + 1, size=S)
    n[rng.random(S) < empty] = 0
    for at in rng.integers(0, S, size=3):      # and in a row, at the ends too
        n[at:at + 5] = 0
    if seed % 2:
        n[0] = n[-1] = 0
    return [int(x) for x in n]


@pytest.mark.parametrize("S", [1, 2, 63, 64, 65, 127, 129, 700, 2048])
@pytest.mark.parametrize("hkv,longest,empty", [(1, 16, 0.3), (3, 40, 0.1), (8, 300, 0.5), (7, 1200, 0.0)])
def test_lengths(device, S, hkv, longest, empty):
    longest = min(longest, max(16, 2_000_000 // (S * hkv)))
    lens = lengths(S, longest, empty, S + hkv) if S > 5 else [16 * longest - 3] * S
    w = wl.custom(lens, hkv, hkv, seed=S, num_pool_blocks=sum((n + 15) // 16 for n in lens) + 1, head_dim=64,
                  partition_size=0 if S % 2 else 64)
    q, k, v = wl.make_host_tensors(w, poison_unused=True)
    print(f"S={S} hkv={hkv} {sum(lens)} tokens", flush=True)
    got = run_attn(w, q, k, v)
    ref = oracle.paged_decode_attn(q, k, v, w.block_tables, w.context_lens, w.scale)
    c = oracle.compare(got, ref)
    assert c["rel_l2"] <= REL_L2 and c["worst_seq_rel_l2"] <= 2 * REL_L2 and abs_error_within_bar(got, ref), c
    assert np.isfinite(wl.bf16_bits_to_f64(got)).all()
    for s in (s for s, n in enumerate(lens) if n == 0):
        assert not got.reshape(w.q_shape())[s].any()
