"""The library's build needs nothing of torch: its link does not wait for the extension module, whose failure is reported
behind it, and where there is no torch the module is left out with a warning."""
from __future__ import annotations

import subprocess
import sys

import pytest

from paper_2412_19829_amd import build


@pytest.fixture
def commands(monkeypatch, tmp_path):
    done = []
    monkeypatch.setattr(build, "OBJ_DIR", str(tmp_path))
    monkeypatch.setattr(build.subprocess, "run", lambda cmd, **kw: done.append(cmd))
    return done


def _links(commands):
    return [c for c in commands if "-shared" in c and build.LIB in c]


def test_a_module_that_does_not_compile(commands, monkeypatch):
    def fails():
        raise subprocess.CalledProcessError(1, "g++")
    monkeypatch.setattr(build, "_build_call", fails)
    with pytest.raises(subprocess.CalledProcessError):
        build.build(force=True)
    assert len(_links(commands)) == 1


def test_without_torch(commands, monkeypatch):
    monkeypatch.setitem(sys.modules, "torch", None)
    with pytest.warns(UserWarning, match="not built"):
        assert build.build(force=True) == build.LIB
    assert len(_links(commands)) == 1 and not any(build.CALL in c for c in commands)


def test_both(commands):
    build.build(force=True)
    assert len(_links(commands)) == 1 and sum(build.CALL in c for c in commands) == 1
