"""The stream-read probe asks for K and V as the stream pass does at D = 128 in bf16, in the assembly that the sources give (no GPU):
whole rows, 1 KiB in a row per load, never 64 bytes of each of 16 tokens."""
import os
import re
import subprocess

from paper_2602_11530_amd import build as pkv_build

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_11530_amd", "csrc")


def test_probe_reads_whole_rows(tmp_path):
    asm = str(tmp_path / "probe.s")
    flags = [f for f in pkv_build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([pkv_build.HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(CSRC, "stream_probe.hip"), "-o", asm],
                          stderr=subprocess.DEVNULL)
    loads = re.findall(r"global_load_dwordx4 [^\n]* nt\b", open(asm).read())
    offsets = [int((re.search(r"offset:(\d+)", load) or [0, 0])[1]) for load in loads]
    assert len(loads) >= 16 and set(offsets) == {0, 1024, 2048, 3072}, loads   # two blocks a turn
