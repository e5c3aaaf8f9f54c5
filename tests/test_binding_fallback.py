"""The package without its binding's native part, or with one of another torch: a warning, and every call through ctypes; and when the build
makes that part anew.  Nothing is launched."""
import importlib.util
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CALLS = """
import warnings
with warnings.catch_warnings(record=True) as caught:
    warnings.simplefilter("always")
    import paper_1609_07061_amd as q
assert any("native part" in str(w.message) for w in caught) == {expected}, [str(w.message) for w in caught]
import torch
x, out = torch.zeros(8, 64), torch.zeros(8, 2, dtype=torch.int32)
for call in (lambda: q.qnn_pack_sign(x, out=out), lambda: q.qnn_binary_gemm(out, out, 64, out=torch.zeros(8, 8, dtype=torch.int32))):
    try:
        call()
    except ValueError as e:
        assert "must be a GPU tensor" in str(e), e
    else:
        raise AssertionError("a CPU tensor was taken")
print("fine")
"""
# as a module of that name that is not there, is not like ours, or was built for something else, whose functions must not be called
MISSING = 'import sys; sys.modules["paper_1609_07061_amd._native"] = None\n'
OTHER = 'import sys, types; m = sys.modules["paper_1609_07061_amd._native"] = types.ModuleType("_native"); {}\n'


@pytest.mark.parametrize("before,expected", [("", False), (MISSING, True), (OTHER.format("m.pack_sign = None"), True),
                                             (OTHER.format('m.BUILT_FOR = "torch 0.1, cpython-27"'), True)])
def test_import(before, expected):
    r = subprocess.run([sys.executable, "-c", before + CALLS.format(expected=expected)], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.endswith("fine\n"), r.stdout + r.stderr


def _build_module(tmp_path, monkeypatch):
    spec = importlib.util.spec_from_file_location("_qnn_build_test", os.path.join(ROOT, "paper_1609_07061_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    monkeypatch.setattr(b, "NATIVE", str(tmp_path / "_native.so"))
    monkeypatch.setattr(b, "NATIVE_STAMP", str(tmp_path / "native.txt"))
    return b


def test_built_anew_for_another_torch(tmp_path, monkeypatch):
    b = _build_module(tmp_path, monkeypatch)
    assert b._binding_stale()
    (tmp_path / "_native.so").write_bytes(b"")
    assert b._binding_stale()  # (nobody knows for which)
    b._build_binding(lambda cmd: (tmp_path / "_native.so").write_bytes(b""))
    assert not b._binding_stale()
    monkeypatch.setattr("torch.__version__", "0.1")
    assert b._binding_stale()


def test_library_is_built_without_a_compiler_for_it(tmp_path, monkeypatch, capfd):
    def no_compiler(cmd):
        raise FileNotFoundError("g++")

    b = _build_module(tmp_path, monkeypatch)
    (tmp_path / "_native.so").write_bytes(b"")
    b._build_binding(no_compiler)
    assert not (tmp_path / "_native.so").exists()  # (one of another source or torch does not stay)
    assert "not built" in capfd.readouterr().err and b._binding_stale()
