"""Loads of the stream pass end at a request's last token, and descriptors come in windows of 64 blocks: shares that end on either side of a
window, a ragged last block in each request with NaN behind it and an unmapped block in each, against fp32 matrix products."""
import numpy as np
import pytest
import torch

from paper_2602_11530_amd import binding as pkv
from paper_2602_11530_amd import workloads as wl

from gpu_util import REL_L2

pytestmark = pytest.mark.gpu
KS, VS = 0.0134, 0.0171


def pool(kv, scale, shape, g, behind):
    """N(0, 1) with NaN in the rows `behind` (block, token)."""
    x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
    x[behind[0], 0, behind[1]] = float("nan")
    return x.to(torch.bfloat16) if kv == "bf16" else (x / scale).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)


def values(kv, scale, rows):
    return rows.float() if kv == "bf16" else rows.view(torch.float8_e4m3fn).float() * scale


@pytest.mark.expects_id_faults
@pytest.mark.parametrize("D,kv,waves", [(64, "bf16", 2048), (64, "fp8", 2048), (128, "bf16", 2048), (128, "fp8", 2048), (256, "bf16", 1024)])
@pytest.mark.parametrize("share,more", [(1, 3), (62, 1900), (63, 0), (64, 0), (64, 1), (65, 700), (127, 1), (129, 2)])
def test_shares_around_a_window(device, id_faults, D, kv, waves, share, more):
    G, S = 2, 12
    total = waves * share + more
    blocks = [total // S] * S
    blocks[0] += total - sum(blocks)
    lens = [16 * n - s for s, n in enumerate(blocks)]   # 16 .. 5 tokens in the last block
    g = torch.Generator(device="cuda")
    g.manual_seed(share * 10 + more)
    ids = torch.randperm(total, generator=g, device="cuda").to(torch.int32)
    width, at = max(blocks), np.cumsum([0] + blocks)
    tables = torch.full((S, width), -1, dtype=torch.int32, device="cuda")
    for s in range(S):
        tables[s, :blocks[s]] = ids[at[s]:at[s + 1]]
    last = [(int(tables[s, blocks[s] - 1]), t) for s in range(S) for t in range(lens[s] - 16 * (blocks[s] - 1), 16)]
    behind = [torch.tensor([x[i] for x in last], dtype=torch.long, device="cuda") for i in (0, 1)]
    q = torch.randn((S, G, D), generator=g, device="cuda").to(torch.bfloat16)
    k, v = (pool(kv, c, (total, 1, 16, D), g, behind) for c in (KS, VS))
    missing = [n // 2 for n in blocks]
    for s in range(S):
        tables[s, missing[s]] = total + 5   # refused: attended over as if it were not there
    lens_d = torch.tensor(lens, dtype=torch.int32, device="cuda")
    shape = pkv.make_shape(S, G, 1, width, total, head_dim=D)
    ws = torch.empty(pkv.pkv_attn_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    out = torch.full_like(q, float("nan"))
    print(f"D={D} {kv} {total} blocks", flush=True)
    if kv == "bf16":
        pkv.paged_decode_attn(q, k, v, tables, lens_d, D ** -0.5, out, shape, ws)
    else:
        pkv.paged_decode_attn_fp8kv(q, k, v, tables, lens_d, D ** -0.5, KS, VS, out, shape, ws)
    torch.cuda.synchronize()
    assert int(id_faults.item()) == S
    for s in range(S):
        keep = torch.ones(blocks[s], dtype=torch.bool, device="cuda")
        keep[missing[s]] = False
        here = tables[s, :blocks[s]][keep].long()
        rows = [values(kv, c, p[here].reshape(-1, D)[:lens[s] - 16]) for p, c in ((k, KS), (v, VS))]
        p = torch.softmax(q[s].float() @ rows[0].t().contiguous() * D ** -0.5, dim=-1)
        ref = p @ rows[1]
        err = (out[s].float() - ref).norm() / ref.norm()
        assert err <= REL_L2, (s, float(err))
