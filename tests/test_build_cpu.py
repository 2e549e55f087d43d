"""CPU-only: what building the library asks for."""
import os
import sys

import pytest

from paper_2504_13989_amd import build


@pytest.fixture
def commands(monkeypatch, tmp_path):
    """the build's commands, recorded instead of run; what they would write exists"""
    ran = []

    def run(cmd, verbose):
        ran.append(cmd)
        open(cmd[cmd.index("-o") + 1], "w").close()

    monkeypatch.setattr(build, "_run", run)
    monkeypatch.setattr(build, "hipcc_path", lambda: "hipcc")
    monkeypatch.setattr(build, "LIB_PATH", str(tmp_path / "librotq.so"))
    monkeypatch.setattr(build, "NATIVE_PATH", str(tmp_path / "_pyrotq.so"))
    return ran


def test_the_library_is_built_without_torch(monkeypatch, commands, capsys):
    monkeypatch.setitem(sys.modules, "torch", None)          # import torch raises ImportError
    assert build.build_library() == build.LIB_PATH
    assert os.path.exists(build.LIB_PATH) and not os.path.exists(build.NATIVE_PATH)
    assert len(commands) == len(build.SOURCES) + 1 and not any("pyrotq" in a for c in commands for a in c)
    assert "left out" in capsys.readouterr().out


def test_the_python_side_comes_after_the_library(commands):
    build.build_library()
    assert os.path.exists(build.LIB_PATH) and os.path.exists(build.NATIVE_PATH)
    assert len(commands) == len(build.SOURCES) + 3
    assert [c[c.index("-o") + 1] for c in commands[-2:]] == [build.LIB_PATH + ".tmp", build.NATIVE_PATH + ".tmp"]
