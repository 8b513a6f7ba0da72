"""The binding's call module is one interpreter's, and optional: what is built, what is left and what goes away."""
import importlib.machinery
import os
import subprocess
import sysconfig

import pytest

from paper_1810_08723_amd import build


@pytest.fixture
def folder(tmp_path, monkeypatch):
    """The build's folder, with the modules of earlier builds in it."""
    suffix = sysconfig.get_config_var("EXT_SUFFIX")
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "CALL", str(tmp_path / os.path.basename(build.CALL)))
    for name in ("_call.so", "_call" + suffix, "_call.cpython-33-other.so"):
        (tmp_path / name).write_text("of an earlier build")
    return tmp_path


def test_only_the_interpreter_that_built_it_finds_it():
    suffix = sysconfig.get_config_var("EXT_SUFFIX")
    assert os.path.basename(build.CALL) == "_call" + suffix and suffix in importlib.machinery.EXTENSION_SUFFIXES
    assert "cpython" in suffix or "abi" in suffix or "pypy" in suffix


def test_the_module_replaces_those_of_earlier_builds(folder):
    build.build_call()
    assert sorted(os.listdir(folder)) == sorted([os.path.basename(build.CALL), "_call.cpython-33-other.so"])
    assert open(build.CALL, "rb").read(4) == b"\x7fELF"


@pytest.mark.parametrize("how", ("no headers", "no compiler", "an error"))
def test_without_it_nothing_old_is_left_and_the_build_goes_on(folder, monkeypatch, capsys, how):
    if how == "no headers":
        monkeypatch.setattr(sysconfig, "get_paths", lambda: {"include": str(folder)})
    elif how == "no compiler":
        monkeypatch.setenv("PATH", "")
    else:
        monkeypatch.setattr(build, "CSRC", str(folder))
    build.build_call()
    assert os.listdir(folder) == ["_call.cpython-33-other.so"] and "ctypes" in capsys.readouterr().err


def test_experimental_builds_leave_it_alone(folder, monkeypatch):
    before = {n: (folder / n).read_text() for n in os.listdir(folder)}
    monkeypatch.setattr(build, "_TAG", "x")
    monkeypatch.setattr(subprocess, "run", None)
    build.build_call()
    assert before == {n: (folder / n).read_text() for n in os.listdir(folder)}
