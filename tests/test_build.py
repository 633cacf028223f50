"""CPU-only: what the build does on a host without a C compiler or Python's headers, which only the optional extension needs."""
import os
import shutil
import sysconfig

import pytest

from paper_2512_16465_amd import build


def test_without_a_c_compiler_or_headers_the_extension_is_left_out(tmp_path, monkeypatch, capsys):
    monkeypatch.setattr(build, "HERE", str(tmp_path))                   # (nothing built is touched)
    monkeypatch.setenv("PATH", str(tmp_path))
    assert build.build_python_calls(force=True) == "" and "ctypes" in capsys.readouterr().out
    monkeypatch.undo()
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert build.build_python_calls(force=True) == "" and "Python.h" in capsys.readouterr().out
    assert os.listdir(tmp_path) == []


def test_a_compile_error_of_the_extension_is_an_error(tmp_path, monkeypatch):
    include = sysconfig.get_paths()["include"]
    if not shutil.which("gcc") or not os.path.exists(os.path.join(include, "Python.h")):
        pytest.skip("needs the C compiler and Python's headers")
    (tmp_path / "pycall.c").write_text("not C")
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "CSRC", str(tmp_path))
    with pytest.raises(RuntimeError):
        build.build_python_calls(force=True)
