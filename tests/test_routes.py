"""tests/routes.py says of a batch what the library does with it (no GPU)."""
import os
import subprocess

import numpy as np

import routes
from paper_2602_11530_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_11530_amd", "csrc")


def test_the_host_chooses_as_routes_says(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    exe = str(tmp_path / "route_check")
    subprocess.check_call([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "-x", "hip", "-I", CSRC,
                           os.path.join(ROOT, "tests", "route_check.cpp"), os.path.join(CSRC, "pkv_api.hip"), "-o", exe],
                          stderr=subprocess.DEVNULL)
    shapes = [(seqs, hkv * G, hkv, dim, tokens, fp8)
              for dim in (64, 128, 256) for G in (1, 2, 5, 8) for hkv in (1, 2, 7, 8)
              for seqs in (1, 4, 5, 8, 9, 31, 32, 33, 63, 64, 65, 128, 256, 257)
              for tokens in (1, 192, 193, 384, 385, 512, 768, 769, 1024, 1025, 2048, 2049, 30000) for fp8 in (0, 1)]
    out = subprocess.run([exe], input="\n".join(" ".join(map(str, s)) for s in shapes), capture_output=True, text=True).stdout.split("\n")
    seen = set()
    for (seqs, hq, hkv, dim, tokens, fp8), line in zip(shapes, out):
        want = routes.leaves_records(seqs * hkv, (tokens + 15) // 16, dim, fp8)
        waves = routes.full_waves(dim) if want else seqs * hkv * routes.group_waves(dim)
        assert line == f"{want:d} {waves}", (seqs, hq, hkv, dim, tokens, fp8)
        seen.add(want)
    assert len(seen) == 2


def test_records_of_a_segment_block_by_block():
    rng = np.random.default_rng(5)
    for dim, hkv in ((64, 1), (128, 3), (256, 2)):
        for lens in ([3000] * 6, [900, 0, 17] * 30, [int(x) for x in rng.integers(0, 9000, 20)], [40000, 1]):
            w = wl.custom(lens, hkv, hkv, seed=1, head_dim=dim)
            nb = [(n + 15) // 16 for n in lens]
            T = hkv * sum(nb)
            W = min(T, routes.full_waves(dim))
            group = np.empty(T, dtype=np.int64)   # of each block of the stream
            for wave in range(W):
                group[wave * T // W:(wave + 1) * T // W] = wave // routes.group_waves(dim)
            want, at = [], 0
            for n in (n for n in nb if n for _ in range(hkv)):
                want.append(len(set(group[at:at + n].tolist())))
                at += n
            assert routes.records(w) == want
