"""What a build needs (nothing is compiled here)."""
import os
import subprocess
import sys

from paper_2411_05289_amd import build


def test_library_builds_without_torch(monkeypatch, tmp_path, capsys):
    """The library is for C programs too: without torch the binding's marshalling is left out, and a stale
    one does not stay behind."""
    stale = tmp_path / "_host.so"
    stale.write_bytes(b"")
    monkeypatch.setattr(build, "HOST", str(stale))
    monkeypatch.setitem(sys.modules, "torch", None)
    monkeypatch.setattr(subprocess, "check_call", lambda cmd: (_ for _ in ()).throw(AssertionError(cmd)))
    assert build.build_host() is None
    assert "torch" in capsys.readouterr().out and not stale.exists()


def test_marshalling_builds_without_a_system_compiler(monkeypatch, tmp_path):
    """Where there is no g++ the compiler that comes with hipcc takes its place."""
    llvm = tmp_path / "llvm" / "bin"
    llvm.mkdir(parents=True)
    clang = llvm / "clang++"
    clang.write_text("#!/bin/sh\n")
    clang.chmod(0o755)
    (tmp_path / "bin").mkdir()
    monkeypatch.setattr(build, "HIPCC", str(tmp_path / "bin" / "hipcc"))
    monkeypatch.setenv("PATH", str(tmp_path / "bin"))
    monkeypatch.delenv("CXX", raising=False)
    monkeypatch.setattr(build, "HOST", str(tmp_path / "_host.so"))
    seen = []

    def compile_(cmd):
        seen.append(cmd[0])
        open(cmd[cmd.index("-o") + 1], "w").close()

    monkeypatch.setattr(subprocess, "check_call", compile_)
    assert build.build_host(verbose=False) == str(tmp_path / "_host.so")
    assert os.path.realpath(seen[0]) == str(clang)
