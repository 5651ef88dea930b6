"""The extension with cola.py's checks is optional: without g++, torch or the headers
libcola.so builds alone, and an extension of an older build does not stay."""
import sys
import sysconfig

import pytest

from paper_2502_10940_amd import build as B


@pytest.fixture
def old_extension(tmp_path, monkeypatch):
    p = tmp_path / "_torch_args.so"
    p.write_bytes(b"old")
    monkeypatch.setattr(B, "ARGS", str(p))
    return p


def test_no_compiler(old_extension, monkeypatch, capsys):
    monkeypatch.setattr(B, "CXX", "no-such-compiler")
    assert B._build_args(False) is False
    assert not old_extension.exists() and "no no-such-compiler" in capsys.readouterr().err


def test_no_torch(old_extension, monkeypatch, capsys):
    for m in ("torch", "torch.utils", "torch.utils.cpp_extension"):
        monkeypatch.setitem(sys.modules, m, None)
    assert B._build_args(False) is False
    assert not old_extension.exists() and "no torch" in capsys.readouterr().err


def test_no_headers(old_extension, monkeypatch, tmp_path, capsys):
    real = sysconfig.get_paths
    monkeypatch.setattr(sysconfig, "get_paths", lambda *a, **k: {**real(*a, **k), "include": str(tmp_path)})
    assert B._build_args(False) is False
    assert not old_extension.exists() and "no Python.h" in capsys.readouterr().err


def test_a_compile_error_is_one(old_extension, monkeypatch):
    monkeypatch.setattr(B, "CXX", "false")
    with pytest.raises(Exception):
        B._build_args(False)
