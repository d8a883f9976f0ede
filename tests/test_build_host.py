"""The build's two products: the C ABI library needs hipcc alone, so it is linked even where the torch node cannot be built."""
import os
import subprocess
import sys

import pytest

from paper_2505_14669_amd import build as b


@pytest.fixture
def linked(monkeypatch, tmp_path):
    """build() with the compilers replaced; the paths it links"""
    outputs = []

    def run(cmd, **kw):
        outputs.append(os.path.basename(cmd[cmd.index("-o") + 1]))
        return subprocess.CompletedProcess(cmd, 0, "")
    monkeypatch.setattr(b, "OBJDIR", str(tmp_path))
    monkeypatch.setattr(b, "_compile", lambda src: (src + ".o", ""))
    monkeypatch.setattr(b.subprocess, "run", run)
    return outputs


def test_library_is_linked_when_the_torch_node_fails_to_compile(monkeypatch, linked):
    def broken():
        raise RuntimeError("g++ failed on nn_autograd.cpp")
    monkeypatch.setattr(b, "_compile_nn", broken)
    with pytest.raises(RuntimeError, match="nn_autograd"):
        b.build()
    assert linked == ["libquartet.so"]


def test_library_is_built_without_torch(monkeypatch, linked):
    monkeypatch.setitem(sys.modules, "torch", None)
    assert b.build() == b.LIB and linked == ["libquartet.so"]


def test_both_are_linked(monkeypatch, linked):
    monkeypatch.setattr(b, "_compile_nn", lambda: ("nn.o", "/lib"))
    b.build()
    assert linked == ["libquartet.so", os.path.basename(b.NN_LIB)]


def test_torch_node_carries_the_interpreters_tag():
    from importlib.machinery import EXTENSION_SUFFIXES
    assert os.path.basename(b.NN_LIB) == "_nn_native" + EXTENSION_SUFFIXES[0] != "_nn_native.so"
