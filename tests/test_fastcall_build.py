"""Building the binding's optional extension: whatever keeps it from being built is no error, and no older build stays behind."""
import os
import shutil
import sysconfig

import pytest

from paper_2108_13191_amd import build


def have_all():
    return any(map(shutil.which, ("gcc", "cc", "amdclang", "clang"))) and os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h"))


@pytest.fixture
def stale(tmp_path, monkeypatch):
    out = tmp_path / "_fastcall.so"
    out.write_text("an older build")
    monkeypatch.setattr(build, "FASTCALL", str(out))
    return out


@pytest.mark.parametrize("missing", ["compiler", "header", "valid source"])
def test_failure_is_no_error_and_leaves_nothing(stale, tmp_path, monkeypatch, capsys, missing):
    if missing == "compiler":
        monkeypatch.setenv("PATH", str(tmp_path))
    elif missing == "header":
        monkeypatch.setattr(sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    else:
        (tmp_path / "fastcall.c").write_text("no C\n")
        monkeypatch.setattr(build, "CSRC", str(tmp_path))
    build.build_fastcall()
    assert not stale.exists()
    assert "through ctypes" in capsys.readouterr().out


def test_built_where_it_can_be(stale):
    if not have_all():
        pytest.skip("no C compiler or no Python.h")
    build.build_fastcall()
    assert stale.read_bytes()[:4] == b"\x7fELF"
    assert os.path.exists(os.path.join(build.HERE, "_fastcall" + sysconfig.get_config_var("EXT_SUFFIX")))          # and by the whole build
