"""What the attention calls launch, walked on the host (no GPU): every write to the workspace lies inside
it, in every layer of a launch, and the reduce pass hears of every segment that several workgroups share and reads all of it once."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_11530_amd", "csrc")


def test_writes_stay_in_the_workspace(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    exe = str(tmp_path / "attn_launch_check")
    subprocess.check_call([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "-x", "hip", "-I", CSRC,
                           os.path.join(ROOT, "tests", "attn_launch_check.cpp"), os.path.join(CSRC, "pkv_api.hip"),
                           "-o", exe], stderr=subprocess.DEVNULL)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and "failures=0" in out.stdout, out.stdout


@pytest.mark.parametrize("source,variants", [("attn_stream", 9), ("attn_stream_large", 6), ("attn_stream_short", 8)])
def test_stream_pass_lds_begins_aligned(tmp_path, source, variants):
    """The stream pass's dynamic LDS follows its static arrays; records and rows in it are accessed 16 bytes at a time."""
    from paper_2602_11530_amd import build as pkv_build
    asm = str(tmp_path / "out.s")
    flags = [f for f in pkv_build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([pkv_build.HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(CSRC, source + ".hip"), "-o", asm],
                          stderr=subprocess.DEVNULL)
    sizes = re.findall(r"\.amdhsa_group_segment_fixed_size (\d+)", open(asm).read())
    assert len(sizes) == variants and all(int(s) % 16 == 0 for s in sizes), sizes
