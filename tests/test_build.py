"""The build's handling of the binding's native calls, which it can do without:
the compile commands are replaced by small ones."""
import os
import subprocess
import sys

import pytest

from paper_2609_39859_amd import build


def _start(monkeypatch, tmp_path, ok):
    """A compile of _fastcall.so in tmp_path that writes its output and then
    succeeds or fails, beside one of an earlier build."""
    target = tmp_path / "_fastcall.so"
    target.write_text("earlier")
    monkeypatch.setattr(build, "FASTCALL", str(target))
    popen = subprocess.Popen

    def compile_(cmd, **kw):
        out = cmd[cmd.index("-o") + 1]
        return popen([sys.executable, "-c", "import sys; open(%r, 'w').write('new'); sys.exit(%d)"
                      % (out, 0 if ok else 1)])
    monkeypatch.setattr(build.subprocess, "Popen", compile_)
    monkeypatch.setattr(build, "build_c_example", lambda verbose: None)
    return target


def test_native_calls_are_installed_with_the_library(monkeypatch, tmp_path):
    target = _start(monkeypatch, tmp_path, True)
    monkeypatch.setattr(build, "_build_lib", lambda path, sources, verbose: path)
    assert build.build() == build.LIB
    assert target.read_text() == "new" and os.listdir(tmp_path) == ["_fastcall.so"]


def test_a_failed_library_leaves_the_earlier_native_calls(monkeypatch, tmp_path):
    target = _start(monkeypatch, tmp_path, True)

    def fails(path, sources, verbose):
        raise RuntimeError("hipcc failed")
    monkeypatch.setattr(build, "_build_lib", fails)
    with pytest.raises(RuntimeError, match="hipcc failed"):
        build.build()
    assert target.read_text() == "earlier" and os.listdir(tmp_path) == ["_fastcall.so"]


@pytest.mark.parametrize("how", ["compile error", "no compiler"])
def test_the_library_is_built_without_native_calls(monkeypatch, tmp_path, capsys, how):
    _start(monkeypatch, tmp_path, False)
    monkeypatch.setattr(build, "_build_lib", lambda path, sources, verbose: path)
    if how == "no compiler":
        def missing(cmd, **kw):
            raise FileNotFoundError("g++")
        monkeypatch.setattr(build.subprocess, "Popen", missing)
    assert build.build() == build.LIB
    assert os.listdir(tmp_path) == [] and "ctypes" in capsys.readouterr().err
