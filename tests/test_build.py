"""The build needs hipcc alone: without a C compiler or Python's headers the library is there, and the binding goes without its native entry."""
import os

import pytest

from paper_2105_04663_amd import build as b


@pytest.fixture
def elsewhere(tmp_path, monkeypatch):
    """A build of nothing, by a compiler that only makes its last argument."""
    hipcc = tmp_path / "hipcc"
    hipcc.write_text('#!/bin/sh\nfor last; do :; done\n: > "$last"\n')
    hipcc.chmod(0o755)
    monkeypatch.setenv("HIPCC", str(hipcc))
    for name, value in (("UNITS", []), ("OBJ", str(tmp_path / "build")), ("LIB", str(tmp_path / "lib.so")), ("CALL", str(tmp_path / "_call.so"))):
        monkeypatch.setattr(b, name, value)
    return tmp_path


@pytest.mark.parametrize("cc", ["/nonexistent/cc", "false"])
def test_without_a_c_compiler(elsewhere, monkeypatch, capfd, cc):
    monkeypatch.setenv("CC", cc)
    (elsewhere / "_call.so").write_text("of another build")
    assert b.build() == str(elsewhere / "lib.so") and os.path.exists(b.LIB)
    assert not os.path.exists(b.CALL)
    assert "native entry was not built" in capfd.readouterr().err
    with pytest.raises((OSError, RuntimeError)):
        b.build(only=["call"])                       # asked for by name


def test_with_one(elsewhere):
    b.build()
    assert os.path.getsize(b.CALL) > 0
