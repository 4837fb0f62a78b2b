"""The build around the compilers: what a missing or older part of the machine costs, with the compilers stood in for."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2512_04226_amd import build as b

ROOT = os.path.dirname(b.PKG)


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


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
@pytest.mark.parametrize("named", ["path", "name on PATH", "link"])
def test_hip_headers_are_found_however_the_compiler_is_named(named, commands, monkeypatch, tmp_path):
    if named == "link":
        os.symlink("/opt/rocm/bin/hipcc", tmp_path / "hipcc")
    monkeypatch.setenv("PATH", "/opt/rocm/bin", prepend=os.pathsep)
    monkeypatch.setattr(b, "HIPCC", {"path": "/opt/rocm/bin/hipcc", "name on PATH": "hipcc", "link": str(tmp_path / "hipcc")}[named])
    b.build_extension(force=True)
    cmd = commands[-1]
    includes = [cmd[i + 1] for i, a in enumerate(cmd) if a == "-isystem"]
    assert any(os.path.exists(os.path.join(d, "hip", "hip_runtime.h")) for d in includes), includes


def test_the_extension_is_built_again_for_another_torch(commands, monkeypatch):
    import torch
    b.build_extension()
    assert len(commands) == 1
    b.build_extension()
    assert len(commands) == 1                   # nothing changed
    monkeypatch.setattr(torch, "__version__", "9.9.9+other")
    b.build_extension()
    assert len(commands) == 2 and any("9.9.9+other" in a for a in commands[-1])
    b.build_extension()
    assert len(commands) == 2


def test_the_extensions_name_and_contents_say_what_it_is_built_for():
    import importlib.machinery

    import torch
    from paper_2512_04226_amd import _fastcall
    assert b.EXT.endswith(importlib.machinery.EXTENSION_SUFFIXES[0])        # the suffix with Python's own tag
    assert _fastcall.__file__ == b.EXT and _fastcall.torch_version == torch.__version__


@pytest.mark.parametrize("before", [
    "sys.modules['paper_2512_04226_amd._fastcall'] = None",                     # not there, or of another Python
    "torch.__version__ += '.other'",                                             # of another torch
    "sys.modules['paper_2512_04226_amd._fastcall'] = types.ModuleType('old')"])  # of before it had a version
def test_calls_go_the_general_way_without_the_extension(before):
    code = """
import sys, types, warnings, torch
%s
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    from paper_2512_04226_amd import api
assert [w for w in seen if "paper_2512_04226_amd.build" in str(w.message)]
try:
    api.matmul(torch.zeros(8, 8, dtype=torch.bfloat16), torch.zeros(8, 8, dtype=torch.bfloat16))
except ValueError as e:
    assert "one GPU" in str(e)
else:
    raise AssertionError("refused nothing")
""" % before
    run = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, cwd=ROOT)
    assert run.returncode == 0, run.stderr


def test_an_unbuilt_tree_says_how_to_build_it(tmp_path):
    pkg = tmp_path / "paper_2512_04226_amd"
    pkg.mkdir()
    for name in ("__init__.py", "api.py", "binding.py"):
        shutil.copy(os.path.join(b.PKG, name), pkg / name)
    run = subprocess.run([sys.executable, "-c", "from paper_2512_04226_amd import api"], capture_output=True, text=True, cwd=tmp_path)
    assert run.returncode != 0 and "libgemm355.so is not built: run" in run.stderr, run.stderr
