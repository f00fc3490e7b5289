"""The calls that a serving program makes, with the sizes it makes them at: what the library's speed is judged on.

A case is one pass through the public entry points of ``binding``:

* ``decode``   the KV side of one decode step of one layer: the new token's rows are appended, then every request attends
               over its whole cache (bf16 or 8-bit pools; the caller's workspace or the library's fixed one)
* ``layers``   the same for several layers, attention of all of them in one call
* ``migrate``  blocks of the K and the V pool leave through a staging image and are installed at other block ids
* ``move``     blocks of the K and the V pool go straight into another instance's pools on the same GPU
* ``preempt``  a request's blocks go to pinned host memory and come back into other block ids

Context lengths belong to the case (so its work is known); the values, the order of the requests and the placement of
their blocks come from the seed.  Values are N(0, 1) in bf16, and 8-bit pools hold N(0, 1) divided by the pool's scale.
"""
import math

import numpy as np
import torch

from paper_2602_11530_amd import binding as pkv

K_SCALE, V_SCALE = 0.0134, 0.0171   # 8-bit pools: 448 of them cover 6 and 7.7 sigma


# ---------------------------------------------------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------------------------------------------------
def _decode(name, seqs, lo, hi, mix="uniform", hq=40, hkv=8, dim=128, block=16, kv="bf16", partition=0, entry="workspace",
            layers=0, lens_seed=1):
    c = {"kind": "layers" if layers else "decode", "seqs": seqs, "lo": lo, "hi": hi, "mix": mix, "hq": hq, "hkv": hkv, "dim": dim,
         "block": block, "kv": kv, "partition": partition, "entry": entry, "layers": layers, "lens_seed": lens_seed}
    return {"name": name, **c} if name else c


def _copy(name, kind, blocks, hkv=8, dim=128, block=16, kv="bf16", pool_blocks=0):
    c = {"kind": kind, "blocks": blocks, "hkv": hkv, "dim": dim, "block": block, "kv": kv, "pool_blocks": pool_blocks or 3 * blocks}
    return {"name": name, **c} if name else c


def listed():
    return [
        # a handful of short answers on a small model shard: nothing but latency
        _decode("tiny_b4", 4, 17, 300, hq=8, hkv=2),
        # one user, one long chain of thought (odd length): interactive latency
        _decode("one_8k", 1, 8191, 8191),
        # a few requests on a model with wide heads and 64-token blocks, through the call that needs no workspace
        _decode("b8_d256_static", 8, 1000, 3000, hq=16, hkv=8, dim=256, block=64, entry="static"),
        # many requests just past their prompt, with short contexts: hundreds of segments, each of a few blocks
        _decode("b512_short", 512, 16, 512),
        # a middling batch on a model with narrow heads and 32-token blocks
        _decode("b32_d64", 32, 500, 6000, hq=32, hkv=8, dim=64, block=32),
        # the served model's ordinary full batch
        _decode("b64_qwen32b", 64, 1024, 8192),
        # the same batch on 8-bit pools
        _decode("b64_fp8", 64, 1024, 8192, kv="fp8"),
        # the long-reasoning batch: lognormal lengths, split-K partitions of 512 tokens
        _decode("b128_longcot", 128, 512, 32768, mix="lognormal", partition=512),
        # the whole KV side of a step over several layers: 70 % reasoning, 30 % answering requests
        _decode("layers6_b24", 24, 1024, 16384, mix="phases", layers=6),
        # a quarter of the full batch is evicted and installed elsewhere, K and V
        _copy("migrate_b16", "migrate", 4675, pool_blocks=14000),
        # one request of 5001 tokens crosses to the answering instance on the same GPU, 8-bit pools
        _copy("move_one_fp8", "move", 313, kv="fp8", pool_blocks=6000),
        # one request of 5001 tokens is preempted to host memory and resumed
        _copy("preempt_one", "preempt", 313, pool_blocks=2000),
    ]


_HEADS = [(40, 8), (32, 8), (16, 8), (28, 4), (10, 2), (8, 2), (8, 8), (8, 1)]   # whole models and their shards


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode"] * 6 + ["layers", "migrate", "move", "preempt"])
    dim = rng.choice([128, 128, 128, 64, 256])
    block = rng.choice([16, 16, 32, 64])
    kv = rng.choice(["bf16", "bf16", "fp8"])
    hq, hkv = rng.choice(_HEADS)
    if kind in ("migrate", "move", "preempt"):
        image = hkv * block * dim * (2 if kv == "bf16" else 1)
        most = (1 << 24) if kind == "preempt" else (3 << 26)
        blocks = _log_int(rng, 4, max(8, min(8000, most // image)))
        return _copy(None, kind, blocks, hkv=hkv, dim=dim, block=block, kv=kv, pool_blocks=3 * blocks + rng.randrange(64))
    layers = rng.randrange(2, 7) if kind == "layers" else 0
    if layers:
        kv = "bf16"                      # the all-layers call takes bf16 pools
    hi = _log_int(rng, 64, 32768)
    lo = max(1, int(hi * rng.uniform(0.05, 1.0)))
    token = 2 * hkv * dim * (2 if kv == "bf16" else 1) * max(layers, 1)
    seqs = _log_int(rng, 1, max(1, min(1024, (3 << 30) // (token * hi))))
    entry = "static" if kv == "bf16" and not layers and seqs * hkv <= 4096 and rng.random() < 0.3 else "workspace"
    partition = rng.choice([0, 0, 0, 512])
    return _decode(None, seqs, lo, hi, hq=hq, hkv=hkv, dim=dim, block=block, kv=kv, partition=partition, entry=entry, layers=layers,
                   lens_seed=rng.randrange(1, 1 << 30))


def _lengths(case):
    rng = np.random.default_rng(case["lens_seed"])
    n, lo, hi = case["seqs"], case["lo"], case["hi"]
    if case["mix"] == "lognormal":
        return np.clip(np.rint(np.exp(rng.normal(math.log(6000.0), 0.8, size=n))), lo, hi).astype(np.int32)
    if case["mix"] == "phases":          # reasoning requests are long, answering ones a quarter of that at most
        reasoning = int(round(0.7 * n))
        return np.concatenate([rng.integers(hi // 4, hi + 1, size=reasoning),
                               rng.integers(lo, hi // 4 + 1, size=n - reasoning)]).astype(np.int32)
    return rng.integers(lo, hi + 1, size=n).astype(np.int32)


def _elem(case):
    return 2 if case["kv"] == "bf16" else 1


def _image_bytes(case):
    return case["hkv"] * case["block"] * case["dim"] * _elem(case)


# ---------------------------------------------------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------------------------------------------------
def _normal(shape, g):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _pool(case, blocks, g, scale):
    """One pool of N(0, 1) values: bf16, or e4m3 bytes of the values divided by the pool's scale."""
    shape = (blocks, case["hkv"], case["block"], case["dim"])
    if case["kv"] == "bf16":
        pool = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    else:
        pool = torch.empty(shape, dtype=torch.uint8, device="cuda")
    step = max(1, (1 << 26) // (shape[1] * shape[2] * shape[3]))
    for b in range(0, blocks, step):
        part = _normal((min(step, blocks - b),) + shape[1:], g)
        if case["kv"] == "bf16":
            pool[b:b + step] = part
        else:
            pool[b:b + step] = (part / scale).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    return pool


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rng = np.random.default_rng(seed)
    if case["kind"] in ("decode", "layers"):
        return _prepare_decode(case, g, rng)
    return _prepare_copy(case, g, rng)


def _prepare_decode(case, g, rng):
    lens = rng.permutation(_lengths(case)).astype(np.int32)
    used = (lens.astype(np.int64) + case["block"] - 1) // case["block"]
    n_pool, width = int(used.sum()), int(used.max())
    ids = rng.permutation(n_pool).astype(np.int32)
    tables = np.full((case["seqs"], width), -1, dtype=np.int32)
    at = 0
    for s, n in enumerate(used):
        tables[s, :n] = ids[at:at + n]
        at += n
    n_layers = max(case["layers"], 1)
    per_layer = []
    for _ in range(n_layers):
        new = [_normal((case["seqs"], case["hkv"], case["dim"]), g).to(torch.bfloat16) for _ in range(2)]
        q = _normal((case["seqs"], case["hq"], case["dim"]), g).to(torch.bfloat16)
        per_layer.append({"q": q, "k_new": new[0], "v_new": new[1], "k_pool": _pool(case, n_pool, g, K_SCALE),
                          "v_pool": _pool(case, n_pool, g, V_SCALE), "out": torch.empty_like(q)})
    shape = pkv.make_shape(case["seqs"], case["hq"], case["hkv"], width, n_pool, head_dim=case["dim"], block_size=case["block"],
                           partition_size=case["partition"])
    state = {"case": case, "layers": per_layer, "tables": torch.from_numpy(tables).cuda(), "lens": torch.from_numpy(lens).cuda(),
             "shape": shape, "scale": 1.0 / math.sqrt(case["dim"])}
    if case["entry"] != "static":
        state["ws"] = torch.empty(pkv.pkv_attn_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    if case["kind"] == "layers":         # the pools of a model do not move between steps
        state["pointers"] = [pkv.pointer_array([layer[x] for layer in per_layer]) for x in ("q", "k_pool", "v_pool", "out")]
    return state


def _prepare_copy(case, g, rng):
    n, n_pool = case["blocks"], case["pool_blocks"]
    ids = rng.permutation(n_pool).astype(np.int32)
    state = {"case": case, "n": n, "bytes": _image_bytes(case), "old": torch.from_numpy(ids[:n].copy()).cuda()}
    state["pools"] = [_pool(case, n_pool, g, s) for s in (K_SCALE, V_SCALE)]
    image = (n,) + tuple(state["pools"][0].shape[1:])
    if case["kind"] == "move":           # another instance's pools, with free blocks of its own
        state["to"] = [_pool(case, n_pool, g, s) for s in (K_SCALE, V_SCALE)]
        state["new"] = torch.from_numpy(rng.permutation(n_pool).astype(np.int32)[:n].copy()).cuda()
    else:                                # free blocks of the same pool
        state["new"] = torch.from_numpy(ids[n:2 * n].copy()).cuda()
        state["staging"] = torch.empty(image, dtype=state["pools"][0].dtype, device="cuda")
    if case["kind"] == "preempt":
        state["host"] = [torch.empty(image, dtype=state["pools"][0].dtype, pin_memory=True) for _ in range(2)]
    return state


# ---------------------------------------------------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------------------------------------------------
def run(state):
    case = state["case"]
    if case["kind"] in ("decode", "layers"):
        return _run_decode(state, case)
    n, size, old, new = state["n"], state["bytes"], state["old"], state["new"]
    if case["kind"] == "move":
        for src, dst in zip(state["pools"], state["to"]):
            pkv.kv_blocks_move(src, old, dst, new, n, size, src.shape[0], dst.shape[0])
        return list(state["to"])
    if case["kind"] == "migrate":
        for pool in state["pools"]:
            pkv.kv_blocks_gather(pool, old, state["staging"], n, size, pool.shape[0])
            pkv.kv_blocks_scatter(state["staging"], pool, new, n, size, pool.shape[0])
        return [*state["pools"], state["staging"]]
    for pool, host in zip(state["pools"], state["host"]):
        pkv.kv_blocks_offload(pool, old, state["staging"], host, n, size, pool.shape[0])
    for pool, host in zip(state["pools"], state["host"]):
        pkv.kv_blocks_reload(host, state["staging"], pool, new, n, size, pool.shape[0])
    return [*state["pools"], *state["host"]]


def _run_decode(state, case):
    tables, lens, shape, scale = state["tables"], state["lens"], state["shape"], state["scale"]
    for layer in state["layers"]:
        if case["kv"] == "fp8":
            pkv.kv_append_fp8(layer["k_new"], layer["v_new"], layer["k_pool"], layer["v_pool"], tables, lens, K_SCALE, V_SCALE, shape)
        else:
            pkv.kv_append(layer["k_new"], layer["v_new"], layer["k_pool"], layer["v_pool"], tables, lens, shape)
    if case["kind"] == "layers":
        pkv.paged_decode_attn_layers(*state["pointers"][:3], tables, lens, scale, state["pointers"][3], shape, state["ws"])
    elif case["kv"] == "fp8":
        pkv.paged_decode_attn_fp8kv(layer["q"], layer["k_pool"], layer["v_pool"], tables, lens, scale, K_SCALE, V_SCALE, layer["out"],
                                    shape, state["ws"])
    elif case["entry"] == "static":
        pkv.paged_decode_attn_static(layer["q"], layer["k_pool"], layer["v_pool"], tables, lens, scale, layer["out"], shape)
    else:
        pkv.paged_decode_attn(layer["q"], layer["k_pool"], layer["v_pool"], tables, lens, scale, layer["out"], shape, state["ws"])
    return [[layer["out"], layer["k_pool"], layer["v_pool"]] for layer in state["layers"]]


# ---------------------------------------------------------------------------------------------------------------------
# What a pass cannot do without, and what its results may differ by
# ---------------------------------------------------------------------------------------------------------------------
def work(case):
    if case["kind"] in ("decode", "layers"):
        lens = _lengths(case).astype(np.int64)
        tokens, seqs, layers = int(lens.sum()), case["seqs"], max(case["layers"], 1)
        row = case["hkv"] * case["dim"]
        kv = 2 * tokens * row * _elem(case)                          # every valid K and V row once, shared by its query group
        new = 2 * seqs * row * (2 + _elem(case))                     # the new rows in, and into their slots
        rows = 2 * seqs * case["hq"] * case["dim"] * 2               # q in, out out
        table = 4 * int(((lens + case["block"] - 1) // case["block"]).sum()) + 4 * seqs
        return {"bytes": layers * (kv + new + rows + table), "flops": layers * 4 * tokens * case["hq"] * case["dim"]}
    image = case["blocks"] * _image_bytes(case)
    passes = {"move": 2, "migrate": 4, "preempt": 4}[case["kind"]]   # reads and writes of each image
    return {"bytes": 2 * passes * image + 2 * 4 * case["blocks"], "flops": 0}


def tolerance(case):
    if case["kind"] in ("decode", "layers"):
        # the output's rounding to bf16 is all that shows: 1.65e-3 of the 2-norm, half a unit in the last place at most
        return {"rel": 6.6e-3, "max": 1.6e-2}
    return "exact"


def exact(case, seed):
    if case["kind"] not in ("decode", "layers"):
        return _exact_copy(case, seed)
    state = prepare(case, seed)
    lens, tables = state["lens"].tolist(), state["tables"].long()
    scale = float(np.float32(state["scale"]))
    group = case["hq"] // case["hkv"]
    result = []
    for layer in state["layers"]:
        k_pool, v_pool = layer["k_pool"], layer["v_pool"]
        for pool, new, pool_scale in ((k_pool, layer["k_new"], K_SCALE), (v_pool, layer["v_new"], V_SCALE)):
            if case["kv"] == "fp8":      # the division is part of the format's definition and happens in fp32
                divisor = torch.full((1,), pool_scale, dtype=torch.float32, device="cuda")
                new = (new.float() / divisor).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
            last = state["lens"].long() - 1
            ids = tables.gather(1, (last // case["block"])[:, None])[:, 0]
            pool[ids, :, last % case["block"]] = new

        def rows(pool, s, pool_scale):
            """[hkv][L][dim] in 64 bits"""
            n = (lens[s] + case["block"] - 1) // case["block"]
            x = pool[tables[s, :n]]
            if case["kv"] == "fp8":
                x = x.view(torch.float8_e4m3fn).float().double() * float(np.float32(pool_scale))
            x = x.double().permute(1, 0, 2, 3).reshape(case["hkv"], -1, case["dim"])
            return x[:, :lens[s]].contiguous()

        out = torch.zeros(layer["q"].shape, dtype=torch.float64, device="cuda")
        for s in range(case["seqs"]):
            q = layer["q"][s].double().view(case["hkv"], group, case["dim"])
            k, v = rows(k_pool, s, K_SCALE), rows(v_pool, s, V_SCALE)
            p = torch.softmax(torch.bmm(q, k.transpose(1, 2).contiguous()) * scale, dim=-1)
            out[s] = torch.bmm(p, v).reshape(case["hq"], case["dim"])
        result.append([out, k_pool, v_pool])
    return result


def _exact_copy(case, seed):
    state = prepare(case, seed)
    old, new = state["old"].long(), state["new"].long()
    if case["kind"] == "move":
        for src, dst in zip(state["pools"], state["to"]):
            dst[new] = src[old]
        return list(state["to"])
    images = [pool[old] for pool in state["pools"]]
    for pool, image in zip(state["pools"], images):
        pool[new] = image
    if case["kind"] == "migrate":
        return [*state["pools"], images[1]]
    return [*state["pools"], *[image.cpu() for image in images]]
