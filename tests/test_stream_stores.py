"""The stream pass's hidden stores, in the assembly that its source gives (no GPU): the loops that send them off do not wait for
them.  The compiler does not know these stores, so a wait for all but n loads that it puts into such a loop, because the loop
reuses a register that a load may still write to, also waits for all stores but the youngest n."""
import os
import re
import subprocess

from paper_2602_11530_amd import build as pkv_build

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_11530_amd", "csrc")


def loops_with_hidden_stores(kernel):
    """(first line, last line, waits) of the innermost loops"""
    at, loops = {}, set()
    for i, line in enumerate(kernel):
        label = re.match(r"(\.LBB\w+):", line)
        if label:
            at[label[1]] = i
        jump = re.search(r"s_c?branch\w*\s+(\.LBB\w+)", line)
        if jump and jump[1] in at:
            loops.add((at[jump[1]], i))
    for a, b in sorted(loops):
        inner = not any(a <= c and d <= b and (c, d) != (a, b) for c, d in loops)
        body = kernel[a:b + 1]
        if inner and any("global_store_dwordx4" in x and "sc1" in x for x in body):
            yield a, b, [int(n) for x in body for n in re.findall(r"vmcnt\((\d+)\)", x)]


def test_store_loops_do_not_wait_for_their_stores(tmp_path):
    asm = str(tmp_path / "attn_stream.s")
    flags = [f for f in pkv_build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([pkv_build.HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(CSRC, "attn_stream.hip"), "-o", asm],
                          stderr=subprocess.DEVNULL)
    kernels = re.findall(r"^(_ZN\S*attn_stream_kernel\S*):(.*?)^\.Lfunc_end", open(asm).read(), re.S | re.M)
    assert len(kernels) == 9
    for name, body in kernels:
        found = list(loops_with_hidden_stores(body.split("\n")))
        assert len(found) >= 7, name   # finished rows in the stream (four copies of it) and behind it, two records
        # three in flight: a record takes up to 9 stores
        assert all(n >= 3 for _, _, waits in found for n in waits), (name, found)
