"""The stream pass's loads and hidden stores, in the assembly that its source gives (no GPU).  The loops that send the stores off
do not wait for them: the compiler does not know these stores, so a wait for all but n loads that it puts into such a loop, because the loop
reuses a register that a load may still write to, also waits for all stores but the youngest n."""
import os
import re
import subprocess

import pytest

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


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """(name, assembly) of every variant"""
    asm = str(tmp_path_factory.mktemp("asm") / "attn_stream.s")
    flags = [f for f in pkv_build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([pkv_build.HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(CSRC, "attn_stream.hip"), "-o", asm],
                          stderr=subprocess.DEVNULL)
    found = re.findall(r"^(_ZN\S*attn_stream_kernel\S*):(.*?)^\.Lfunc_end", open(asm).read(), re.S | re.M)
    assert len(found) == 9
    return found


def test_small_blocks_go_out_before_the_last_has_arrived(kernels):
    """e4m3 at D = 64: K of a block is waited for with its four V loads and the five of the next block out."""
    waits = [max(int(n) for n in re.findall(r"vmcnt\((\d+)\)", body)) for name, body in kernels if "ILi64ELb1E" in name]
    assert waits == [9]


def test_store_loops_do_not_wait_for_their_stores(kernels):
    for name, body in kernels:
        found = list(loops_with_hidden_stores(body.split("\n")))
        assert len(found) >= 7, name   # finished rows in the stream (four copies of it) and behind it, two records
        # three in flight: a record takes up to 9 stores
        assert all(n >= 3 for _, _, waits in found for n in waits), (name, found)
