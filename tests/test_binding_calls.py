"""The module that takes the arguments of the serving loop's calls apart agrees with ctypes: same status for the same arguments, and
what it leaves alone is converted or refused by ctypes as before (no GPU: calls that end before a launch)."""
import ctypes
import os
import shutil
import subprocess
import sys

import pytest

from paper_2602_11530_amd import binding as pkv


class Buffer:
    """As much of a tensor as the binding looks at."""

    def __init__(self, address, n=0):
        self.address, self.n = address, n

    def data_ptr(self):
        return self.address

    def numel(self):
        return self.n

    def element_size(self):
        return 1


class Side:
    cuda_stream = 48


T, ODD = Buffer(1 << 20), Buffer((1 << 20) + 2)
SHAPE, BAD, EMPTY = pkv.make_shape(4, 8, 2, 19, 128), pkv.make_shape(4, 8, 3, 19, 128), pkv.make_shape(0, 8, 2, 19, 128)
WS = Buffer(1 << 20, 64)


def status(fn, *args):
    try:
        fn(*args)
    except pkv.PkvError as e:
        return e.status
    return pkv.PKV_OK


@pytest.fixture(params=["module", "ctypes"])
def path(request, monkeypatch):
    pkv.lib()
    if request.param == "ctypes":
        monkeypatch.setattr(pkv, "_call", pkv._ByCtypes())


@pytest.mark.parametrize("stream", [0, 16, Side()])
def test_statuses(path, stream):
    a, c = (T,) * 5, (T, T, T)
    assert status(pkv.kv_append, *a, T, EMPTY, stream) == pkv.PKV_OK
    assert status(pkv.kv_append, *a, T, BAD, stream) == pkv.PKV_ERR_SHAPE
    assert status(pkv.kv_append, *a, None, SHAPE, stream) == pkv.PKV_ERR_NULL
    assert status(pkv.kv_append, *a, ODD, SHAPE, stream) == pkv.PKV_ERR_ALIGN
    assert status(pkv.kv_append_fp8, *a, T, 0.5, -1.0, SHAPE, stream) == pkv.PKV_ERR_SHAPE
    assert status(pkv.kv_append_fp8, *a, T, 0.5, 1.0, EMPTY, stream) == pkv.PKV_OK
    assert status(pkv.paged_decode_attn, *a, 0.1, T, SHAPE, WS, stream) == pkv.PKV_ERR_WORKSPACE
    assert status(pkv.paged_decode_attn, *a, 0.1, T, SHAPE, None, stream) == pkv.PKV_ERR_WORKSPACE
    assert status(pkv.paged_decode_attn, *a, 0.1, None, EMPTY, None, stream) == pkv.PKV_OK
    assert status(pkv.paged_decode_attn_fp8kv, *a, 0.1, 0.0, 1.0, T, EMPTY, None, stream) == pkv.PKV_ERR_SHAPE
    assert status(pkv.paged_decode_attn_fp8kv, *a, 0.1, 1.0, 1.0, T, SHAPE, WS, stream) == pkv.PKV_ERR_WORKSPACE
    assert status(pkv.paged_decode_attn_static, *a, 0.1, T, BAD, stream) == pkv.PKV_ERR_SHAPE
    for fn in (pkv.kv_blocks_gather, pkv.kv_blocks_scatter):
        assert status(fn, *c, 0, 64, 9, stream) == pkv.PKV_OK
        assert status(fn, *c, 4, 40, 9, stream) == pkv.PKV_ERR_ALIGN
        assert status(fn, *c, -1, 64, 9, stream) == pkv.PKV_ERR_SHAPE
    assert status(pkv.kv_blocks_move, *c, T, 4, 64, -1, 9, stream) == pkv.PKV_ERR_SHAPE
    assert status(pkv.kv_blocks_move, *c, None, 4, 64, 9, 9, stream) == pkv.PKV_ERR_NULL
    assert status(pkv.kv_blocks_offload, *c, T, 0, 64, 9, stream) == pkv.PKV_OK
    assert status(pkv.kv_blocks_reload, T, *c, 4, 40, 9, stream) == pkv.PKV_ERR_ALIGN


def test_what_the_module_leaves_alone(path):
    a = (T,) * 5
    assert status(pkv.paged_decode_attn, *a, 1, T, SHAPE, WS, 0) == pkv.PKV_ERR_WORKSPACE      # a whole number for the scale
    assert status(pkv.kv_blocks_gather, T, T, T, True, 40, 9, 0) == pkv.PKV_ERR_ALIGN
    assert status(pkv.kv_blocks_gather, T, T, T, 1 << 64, 40, 9, 0) == pkv.PKV_ERR_ALIGN        # 0 in 64 bits, as ctypes has it
    with pytest.raises(ctypes.ArgumentError):
        pkv.kv_blocks_gather(T, T, T, 4.0, 64, 9, 0)
    with pytest.raises(TypeError):
        pkv.kv_append(*a, T, None, 0)
    with pytest.raises(TypeError):
        pkv.paged_decode_attn(*a, None, T, SHAPE, WS, 0)
    with pytest.raises(AttributeError):
        pkv.kv_append(*a, 16, SHAPE, 0)
    assert pkv.kv_append(*a, context_lens=T, shape=EMPTY, stream=0) is None


@pytest.mark.parametrize("error", [KeyboardInterrupt, MemoryError, RuntimeError, ValueError])
@pytest.mark.parametrize("where", ["data_ptr", "numel", "cuda_stream"])
def test_other_exceptions_reach_the_caller(path, error, where):
    """One that is raised while the arguments are taken apart and is not about their kind: once, and not swallowed."""
    raised = []

    def fail(self):
        if raised:
            return 64   # an interrupt comes once
        raised.append(1)
        raise error("once")
    bad = type("Bad", (Buffer,), {where: property(fail) if where == "cuda_stream" else fail})(1 << 20, 64)
    buffer, stream = (T, bad) if where == "cuda_stream" else (bad, 0)
    with pytest.raises(error, match="once"):
        pkv.paged_decode_attn(T, T, T, T, T, 0.1, T, EMPTY, buffer, stream)


CALLS = """
import ctypes
from {package} import binding as pkv
t = type("Buffer", (), {{"data_ptr": lambda self: 1 << 20}})()
pkv.kv_blocks_gather(t, t, t, 0, 64, 9, 0)
try:
    pkv.kv_blocks_gather(t, t, t, 4, 40, 9, 0)
except pkv.PkvError as e:
    assert e.status == pkv.PKV_ERR_ALIGN
else:
    assert False
print("called")
"""


@pytest.mark.parametrize("module", [None, b"not for this interpreter"])
def test_without_the_module(tmp_path, module):
    """Every call goes by ctypes where the module was not built, or is no module to this interpreter."""
    package = os.path.dirname(pkv.__file__)
    copy = tmp_path / "pkv_copy"
    copy.mkdir()
    for name in ("__init__.py", "binding.py", "workloads.py"):
        shutil.copy(os.path.join(package, name), copy)
    os.symlink(pkv.LIB_PATH, copy / "libpkv.so")
    if module:
        (copy / "_pkv_call.so").write_bytes(module)
    run = subprocess.run([sys.executable, "-c", CALLS.format(package="pkv_copy")], cwd=tmp_path, capture_output=True, text=True)
    assert run.returncode == 0 and "called" in run.stdout, run.stderr
