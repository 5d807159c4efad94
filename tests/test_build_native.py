"""The native call path is optional: a machine without a host compiler, or without
torch's or Python's headers, still builds the library."""
import sysconfig

import pytest
import torch

from paper_2402_18008_amd import build


@pytest.mark.parametrize("missing", ["compiler", "torch headers", "Python headers"])
def test_left_out_where_it_cannot_be_built(monkeypatch, tmp_path, capsys, missing):
    old = tmp_path / "_native.so"
    old.write_bytes(b"built against another libhomog")
    monkeypatch.setattr(build, "NATIVE", str(old))
    monkeypatch.setattr(build, "_run", lambda cmd, what, verbose: pytest.fail("compiled"))
    if missing == "compiler":
        monkeypatch.setattr(build.shutil, "which", lambda name: None)
    elif missing == "torch headers":
        monkeypatch.setattr(torch, "__file__", str(tmp_path / "torch" / "__init__.py"))
    else:
        monkeypatch.setattr(sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert build.build_native() is None
    assert not old.exists()
    assert "_native.so is not built" in capsys.readouterr().err
