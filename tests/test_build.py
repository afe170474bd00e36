"""What a build needs and leaves behind: hipcc alone makes the library, whatever the binding's native calls lack, and nothing
of an earlier build stays beside it."""
import subprocess
import sys

import pytest

from paper_2605_13907_amd import build as M


@pytest.fixture
def place(monkeypatch, tmp_path):
    """A build into tmp_path, where an earlier one has left both files, with a hipcc that only writes its output."""
    def tool(name, body):
        path = tmp_path / name
        path.write_text("#!/bin/sh\n" + body)
        path.chmod(0o755)
        return str(path)

    writes = 'while [ "$1" != "-o" ]; do shift; done\necho new > "$2"\n'
    for attr, name in (("LIB", "lib.so"), ("FAST", "fast.so")):
        (tmp_path / name).write_text("old\n")
        monkeypatch.setattr(M, attr, str(tmp_path / name))
    monkeypatch.setenv("HIPCC", tool("hipcc", writes))
    monkeypatch.setenv("CXX", tool("cxx", writes))
    return tmp_path, monkeypatch, tool


def state(tmp_path):
    return [(tmp_path / n).read_text().strip() if (tmp_path / n).exists() else None for n in ("lib.so", "fast.so")]


def test_both(place):
    M.build(verbose=False)
    assert state(place[0]) == ["new", "new"]


@pytest.mark.parametrize("lacks", ["compiler", "torch", "Python.h"])
def test_library_alone(place, capsys, lacks):
    tmp_path, monkeypatch, _ = place
    if lacks == "compiler":
        monkeypatch.setenv("CXX", "/nowhere/g++")
    elif lacks == "torch":
        import torch.utils
        monkeypatch.setitem(sys.modules, "torch.utils.cpp_extension", None)
        monkeypatch.delattr(torch.utils, "cpp_extension", raising=False)
    else:
        monkeypatch.setattr(M.sysconfig, "get_paths", lambda: {"include": "/nowhere"})
    M.build()
    assert state(tmp_path) == ["new", None]
    assert "native calls are not built" in capsys.readouterr().out


@pytest.mark.parametrize("fails,left", [("CXX", ["new", None]), ("HIPCC", [None, "new"])])
def test_a_step_that_fails(place, fails, left):
    tmp_path, monkeypatch, tool = place
    monkeypatch.setenv(fails, tool("failing", "exit 1\n"))
    with pytest.raises(subprocess.CalledProcessError):
        M.build(verbose=False)
    assert state(tmp_path) == left
