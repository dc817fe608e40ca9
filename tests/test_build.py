"""What build() makes and in which order (CPU; no compiler runs): the library
for C programs needs neither torch nor g++."""

import os
import types

import pytest

from paper_2604_08706_amd import build as b


@pytest.fixture
def commands(tmp_path, monkeypatch):
    """Commands that build() would run; each makes its output file.  fail names
    a program that is not found."""
    ran = types.SimpleNamespace(list=[], fail=None)

    def run(cmd, **_):
        if os.path.basename(cmd[0]) == ran.fail:
            raise FileNotFoundError(cmd[0])
        ran.list.append(cmd)
        open(cmd[cmd.index("-o") + 1], "w").close()
        return types.SimpleNamespace(returncode=0, stdout="", stderr="")

    monkeypatch.setattr(b.subprocess, "run", run)
    monkeypatch.setattr(b, "hipcc", lambda: "/opt/rocm/bin/hipcc")
    monkeypatch.setattr(b, "OBJDIR", str(tmp_path / "_build"))
    monkeypatch.setattr(b, "LIB", str(tmp_path / "librbpolicy.so"))
    monkeypatch.setattr(b, "MARSHAL", str(tmp_path / "_marshal.so"))
    return ran


def test_both_libraries_are_built(commands):
    assert b.build(verbose=False) == b.LIB
    assert os.path.exists(b.LIB) and os.path.exists(b.MARSHAL)


def test_the_library_is_built_without_torch(commands, monkeypatch, capsys):
    import importlib.util

    monkeypatch.setattr(importlib.util, "find_spec", lambda name: None)
    b.build(verbose=False)
    assert os.path.exists(b.LIB) and not os.path.exists(b.MARSHAL)
    assert not any(cmd[0] == "g++" for cmd in commands.list)
    assert "torch is not installed" in capsys.readouterr().err


def test_without_gxx_the_library_is_in_place_and_the_failure_is_raised(commands):
    commands.fail = "g++"
    with pytest.raises(FileNotFoundError):
        b.build(verbose=False)
    assert os.path.exists(b.LIB) and not os.path.exists(b.MARSHAL)
