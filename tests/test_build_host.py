"""The C library stands without torch's headers and without the binding's host module; the binding works without the latter."""
import os
import sys

import pytest

import paper_2512_13368_amd as package
from paper_2512_13368_amd import binding as B
from paper_2512_13368_amd import build


def test_library_is_linked_when_the_host_module_does_not_build(monkeypatch, tmp_path):
    monkeypatch.setattr(build, "SOURCES", {"probe.hip": []})  # (one file: what is linked does not matter here)
    monkeypatch.setattr(build, "OBJ_DIR", str(tmp_path / "obj"))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libblossom.so"))
    monkeypatch.setattr(build, "FASTCALL", str(tmp_path / "_fastcall.so"))
    monkeypatch.setattr(build, "fastcall_command", lambda obj: ["false"])
    with pytest.raises(RuntimeError, match="fastcall.cpp"):
        build.build_all()
    assert os.path.exists(build.LIB) and not os.path.exists(build.FASTCALL)


def test_binding_without_the_host_module(monkeypatch):
    torch = pytest.importorskip("torch")
    monkeypatch.setattr(B, "_fast", None)
    monkeypatch.delattr(package, "_fastcall", raising=False)
    monkeypatch.setitem(sys.modules, package.__name__ + "._fastcall", None)  # (importing it raises ImportError)
    p = B.Params(1, 1, 8, 8, 8, 1, 1)
    with pytest.warns(RuntimeWarning, match="_fastcall"), pytest.raises(ValueError, match="^Q: expected contiguous cuda tensor"):
        B.select_blocks(p, torch.zeros(1, 1, 8, 8), torch.zeros(1, 1, 8, 8), torch.zeros(1, dtype=torch.int32))
    assert B.fastcall() is B.PYTHON_PATH
