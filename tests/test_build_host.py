"""The C library stands without torch's headers and without the binding's host module; the binding works without the latter."""
import os
import subprocess
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


def test_loads_to_lds_leave_m0_to_the_compiler(tmp_path):
    # m0 is the compiler's: it keeps no promise about a value of its own there across assembly that changes it, and says so
    src = tmp_path / "probe.hip"
    src.write_text(f'#include "{build.CSRC}/mfma_common.h"\n'
                   'using namespace blossom;\n'
                   '__global__ void probe(const char *from, uint4 *to) {\n'
                   '  __shared__ uint4 rows[128];\n'
                   '  mfma::load_to_lds(from, threadIdx.x * 16u, threadIdx.x * 16u, __builtin_amdgcn_readfirstlane(mfma::lds_address(rows)));\n'
                   '  mfma::arrived_all<0>();\n'
                   '  to[threadIdx.x] = rows[threadIdx.x + 64];\n'
                   '}\n')
    out = tmp_path / "probe.s"
    r = subprocess.run([build._hipcc(), *build.COMMON, "--cuda-device-only", "-S", str(src), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    assert "reserved" not in r.stderr, r.stderr
    text = out.read_text()
    assembly = text[text.index("ASMSTART"):text.index("ASMEND")]
    assert "global_load_lds" in assembly and "m0" not in assembly and text.count("s_mov_b32 m0") == 1, text
