"""The build on the CPU: the C library is built whether or not the binding's
short path, which needs torch's headers, can be."""
import os
import subprocess
import types

import pytest

from paper_1302_5586_amd import build as b


@pytest.fixture
def fake(tmp_path, monkeypatch):
    """A build of no sources whose compilers are replaced: commands are
    recorded, the linker writes its output, g++ fails."""
    ran = []

    def run(cmd, **kw):
        ran.append(cmd)
        if cmd[0] == "g++":
            return types.SimpleNamespace(returncode=1, stdout="", stderr="no torch headers\n")
        with open(cmd[cmd.index("-o") + 1], "w") as f:
            f.write("library")
        return types.SimpleNamespace(returncode=0, stdout="", stderr="")

    monkeypatch.setattr(subprocess, "run", run)
    monkeypatch.setattr(b, "_jobs", lambda: [("x.cpp", "", [])])
    monkeypatch.setattr(b, "_compile", lambda *a, **k: "x.o")
    monkeypatch.setattr(b, "check_resources", lambda *a: None)
    for name in ("LIB", "FASTCALL", "OBJDIR"):
        monkeypatch.setattr(b, name, str(tmp_path / name.lower()))
    return ran


def test_library_without_the_short_path(fake, capfd):
    with open(b.FASTCALL, "w") as f:
        f.write("of older sources")
    assert b.build(out=b.LIB) == b.LIB and os.path.exists(b.LIB)
    assert any(c[0] == "g++" for c in fake)
    assert not os.path.exists(b.FASTCALL)
    assert "short path is not built" in capfd.readouterr().err


@pytest.mark.parametrize("defines", [[], ["-DPF_CHUNK=4"]])
def test_variants_leave_the_short_path_alone(fake, tmp_path, defines):
    with open(b.FASTCALL, "w") as f:
        f.write("kept")
    out = str(tmp_path / "variant.so")
    assert b.build(out=out, defines=defines) == out and os.path.exists(out)
    assert not any(c[0] == "g++" for c in fake)
    assert open(b.FASTCALL).read() == "kept"
