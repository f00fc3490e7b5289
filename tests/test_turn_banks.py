"""Where K lies in LDS while it is turned (no GPU): a place for every piece, and no bank conflicts."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_no_bank_conflicts(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    exe = str(tmp_path / "turn_banks_check")
    subprocess.check_call([hipcc, "-O1", "--offload-arch=gfx950", "-x", "hip", "-I",
                           os.path.join(ROOT, "paper_2602_11530_amd", "csrc"),
                           os.path.join(ROOT, "tests", "turn_banks_check.cpp"), "-o", exe], stderr=subprocess.DEVNULL)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
