"""The build around the compilers: what a missing or older part of the machine costs, with the compilers stood in for."""
import os
import subprocess

import pytest

from paper_2512_04226_amd import build as b


@pytest.fixture
def commands(tmp_path, monkeypatch):
    """Every command of the build instead of its run: recorded, and its output file made."""
    ran = []

    def run(cmd, **kwargs):
        ran.append(cmd)
        open(cmd[cmd.index("-o") + 1], "w").close()
        return subprocess.CompletedProcess(cmd, 0, "", "")
    monkeypatch.setattr(b.subprocess, "run", run)
    monkeypatch.setattr(b, "OBJ", str(tmp_path / "obj"))
    monkeypatch.setattr(b, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setattr(b, "EXT", str(tmp_path / "ext.so"))
    return ran


def test_the_library_is_linked_where_the_extension_cannot_be_built(commands, monkeypatch, capsys):
    def fails(force=False):
        raise ImportError("no torch here")
    monkeypatch.setattr(b, "build_extension", fails)
    assert b.build(force=True) == b.LIB and os.path.exists(b.LIB)
    assert any("-shared" in c for c in commands)
    assert "no torch here" in capsys.readouterr().err
    with pytest.raises(ImportError):
        b.build(force=True, strict=True)
