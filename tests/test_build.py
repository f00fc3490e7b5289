"""What is built where: the libraries need no Python headers, and the module's name says which interpreter it is for."""
import os
import subprocess
import sys
import sysconfig

import pytest

from paper_2602_11530_amd import build as pkv_build


@pytest.fixture
def built(tmp_path, monkeypatch):
    """Records what build() compiles; pkv_call.cpp does not compile without the headers."""
    outputs = []

    def compile_(cmd, out, verbose):
        if any(x.endswith("pkv_call.cpp") for x in cmd) and not os.path.exists(os.path.join(cmd[cmd.index("-I") + 1], "Python.h")):
            raise subprocess.CalledProcessError(1, cmd)
        outputs.append(out)
        return out
    monkeypatch.setattr(pkv_build, "_compile", compile_)
    monkeypatch.setattr(pkv_build, "CALL", str(tmp_path / os.path.basename(pkv_build.CALL)))
    return outputs


def test_without_python_headers(built, tmp_path, monkeypatch):
    monkeypatch.setattr(sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    with open(pkv_build.CALL, "w"):
        pass
    assert pkv_build.build(verbose=False) == pkv_build.LIB
    assert set(built) == {pkv_build.LIB, pkv_build.SCHED_LIB, pkv_build.DRIVER}
    assert not os.path.exists(pkv_build.CALL)   # none of an earlier build next to a new library


def test_the_module_comes_last(built):
    pkv_build.build(verbose=False)
    assert built[-1] == pkv_build.CALL and set(built[:-1]) == {pkv_build.LIB, pkv_build.SCHED_LIB, pkv_build.DRIVER}


def test_the_module_is_for_this_interpreter():
    name = os.path.basename(pkv_build.CALL)
    assert name == "_pkv_call" + sysconfig.get_config_var("EXT_SUFFIX") != "_pkv_call.so"
    assert sys.implementation.name in name
