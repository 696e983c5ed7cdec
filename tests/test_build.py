"""CPU-only checks of the build's bookkeeping: compilers are stand-ins that leave a file behind."""
import os
import subprocess

import pytest

from paper_2412_07752_amd import build as b


@pytest.fixture
def tree(monkeypatch, tmp_path):
    """An empty source tree of two units; calls of the linker are recorded."""
    csrc, include, calls = tmp_path / "csrc", tmp_path / "include", []
    csrc.mkdir(), include.mkdir()
    for f in (csrc / "a.hip", csrc / "b.hip", csrc / "c.h", include / "flashrnn.h"):
        f.write_text("")
    for name, value in (("CSRC", str(csrc)), ("INCLUDE", str(include)), ("OUT", str(tmp_path / "libflashrnn.so"))):
        monkeypatch.setattr(b, name, value)

    def compile(src, obj, extra=()):
        with open(obj, "w"):
            return ""

    def link(cmd):
        calls.append(cmd)
        with open(cmd[cmd.index("-o") + 1], "w"):
            return 0

    monkeypatch.setattr(b, "_compile", compile)
    monkeypatch.setattr(subprocess, "check_call", link)
    return calls


def test_the_library_is_built_without_the_python_binding(tree, monkeypatch):
    """hipcc alone builds the C ABI: no g++, no Python or torch headers."""
    def binding(force=False):
        raise RuntimeError("no Python.h")

    monkeypatch.setattr(b, "build_binding", binding)
    with pytest.warns(RuntimeWarning, match="no Python.h"):
        out = b.build()
    assert os.path.exists(out) and len(tree) == 1


def test_objects_newer_than_the_library_are_linked(tree, monkeypatch):
    """A build that compiled but did not get to linking must not leave an older library in place for good."""
    monkeypatch.setattr(b, "build_binding", lambda force=False: None)
    out = b.build()
    b.build()
    assert len(tree) == 1   # (nothing to do)
    os.utime(out, (1, 1))
    b.build()
    assert len(tree) == 2
