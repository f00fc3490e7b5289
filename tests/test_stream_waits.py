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
def assembly(tmp_path_factory):
    text = []
    flags = [f for f in pkv_build.FLAGS if f not in ("-fPIC", "-shared")]
    for source in ("attn_stream", "attn_stream_large", "attn_stream_short"):
        asm = str(tmp_path_factory.mktemp("asm") / (source + ".s"))
        subprocess.check_call([pkv_build.HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(CSRC, source + ".hip"), "-o", asm],
                              stderr=subprocess.DEVNULL)
        text.append(open(asm).read())
    return text


@pytest.fixture(scope="module")
def kernels(assembly):
    """(name, assembly) of every variant"""
    found = [k for text in assembly for k in re.findall(r"^(_ZN\S*attn_stream_kernel\S*):(.*?)^\.Lfunc_end", text, re.S | re.M)]
    assert len(found) == 23
    return found


@pytest.mark.parametrize("dim", [64, 128, 256])
def test_short_launches_of_layers_carry_nothing_for_the_chain(assembly, dim):
    """Where each segment has a workgroup the kernel is as for one layer: it saves no scalar registers for layers to come."""
    spills = {name: int(n) for text in assembly
              for name, n in re.findall(r"\.name:\s+(\S*attn_stream_kernel\S*).*?\.sgpr_spill_count:\s+(\d+)", text, re.S)}
    late = "ELb1E" if dim == 128 else "ELb0E"
    one = [n for name, n in spills.items() if f"ILi{dim}ELb0ENS_8OneLayer{late}" in name]
    layers = [n for name, n in spills.items() if f"ILi{dim}ELb0ENS_10AttnLayers{late}" in name]
    assert len(one) == len(layers) == 1 and layers[0] <= one[0] + 8, (one, layers)


def test_small_blocks_go_out_before_the_last_has_arrived(kernels):
    """e4m3 at D = 64: K of a block is waited for with its four V loads and the five of the next block out."""
    waits = {name: max(int(n) for n in re.findall(r"vmcnt\((\d+)\)", body)) for name, body in kernels if "ILi64ELb1E" in name}
    assert len(waits) == 2 and set(waits.values()) == {9}, waits


def test_store_loops_do_not_wait_for_their_stores(kernels):
    for name, body in kernels:
        found = list(loops_with_hidden_stores(body.split("\n")))
        assert len(found) >= 5, name   # finished rows in the stream (four copies of it) and behind it
        # three in flight: a record takes up to 9 stores
        assert all(n >= 3 for _, _, waits in found for n in waits), (name, found)
