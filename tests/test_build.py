"""CPU-only checks of the build's bookkeeping: compilers are stand-ins that leave a file behind."""
import os
import subprocess
import sysconfig

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


def test_the_binding_is_built_anew_for_another_torch(tree, monkeypatch, tmp_path):
    """The file's time says nothing of the headers it was compiled with; what has no ABI tag, or cannot be built again, does not stay."""
    import torch
    made = []

    def compiler(cmd, **kw):
        made.append(cmd)
        with open(cmd[cmd.index("-o") + 1], "w") as f:
            f.write([a for a in cmd if a.startswith("-DFLASHRNN_BUILT_FOR=")][0].split('"')[1] + "\0")
        return subprocess.CompletedProcess(cmd, 0, "")

    monkeypatch.setattr(b, "HERE", str(tmp_path))
    monkeypatch.setattr(subprocess, "run", compiler)
    (tmp_path / "csrc" / "flashrnn_binding.cpp").write_text("")
    (tmp_path / "_flashrnn_binding.so").write_text("")
    out = b.build_binding()
    assert os.path.basename(out) == "_flashrnn_binding" + sysconfig.get_config_var("EXT_SUFFIX") and not (tmp_path / "_flashrnn_binding.so").exists()
    b.build_binding()
    assert len(made) == 1
    monkeypatch.setattr(torch, "__version__", "99.0")
    b.build_binding()
    b.build_binding()
    assert len(made) == 2
    monkeypatch.setattr(torch, "__version__", "99.1")
    monkeypatch.setattr(subprocess, "run", lambda cmd, **kw: subprocess.CompletedProcess(cmd, 1, "no Python.h"))
    with pytest.raises(RuntimeError, match="no Python.h"):
        b.build_binding()
    assert not os.path.exists(out)


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
