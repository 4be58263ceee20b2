"""The build: the library does not depend on what only the optional tensor check needs."""
import os
import subprocess

import pytest

from paper_2510_25979_amd import build


@pytest.fixture
def targets(monkeypatch, tmp_path):
    monkeypatch.setattr(build, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setattr(build, "ARG", str(tmp_path / "arg.so"))
    monkeypatch.setattr(build, "_lib_command", lambda: ["touch", build.LIB])
    monkeypatch.setattr(build, "_arg_command", lambda: ["touch", build.ARG])


def _no_torch():
    raise ImportError("no torch here")


@pytest.mark.parametrize("command", [_no_torch, lambda: ["no-such-compiler"], lambda: ["false"]],
                         ids=["no torch", "no compiler", "no headers"])
@pytest.mark.parametrize("force", [True, False])
def test_the_library_is_built_where_the_tensor_check_cannot_be(targets, monkeypatch, capsys, command, force):
    monkeypatch.setattr(build, "_arg_command", command)
    open(build.ARG, "w").close()
    os.utime(build.ARG, (0, 0))            # of older sources
    assert build.build(force=force) == build.LIB and os.path.exists(build.LIB)
    assert not os.path.exists(build.ARG) and "checked in Python" in capsys.readouterr().err


def test_what_is_up_to_date_is_left_alone(targets, monkeypatch):
    assert build.stale()
    build.build(force=False)
    assert os.path.exists(build.LIB) and os.path.exists(build.ARG) and not build.stale()
    monkeypatch.setattr(build, "_lib_command", lambda: ["false"])
    monkeypatch.setattr(build, "_arg_command", _no_torch)
    assert build.build(force=False) == build.LIB and os.path.exists(build.ARG)


def test_a_library_that_does_not_compile_is_an_error(targets, monkeypatch):
    monkeypatch.setattr(build, "_lib_command", lambda: ["false"])
    with pytest.raises(subprocess.CalledProcessError):
        build.build()
