"""The build where the optional part of it cannot be built (compilers replaced by programs that do nothing or fail)."""
import os

import pytest

from paper_2310_05218_amd import build


@pytest.mark.parametrize("broken", ["compiler", "no compiler", "torch"])
def test_library_is_built_without_the_binding(monkeypatch, tmp_path, capsys, broken):
    stale = tmp_path / "_swnative.so"
    stale.write_bytes(b"of an older build")
    monkeypatch.setattr(build, "BINDING", str(stale))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libswconv.so"))
    monkeypatch.setattr(build, "PKG", str(tmp_path / "package"))        # (the folder of the objects is beside it)
    monkeypatch.setenv("HIPCC", "true")
    if broken == "torch":
        def no_torch(verbose):
            raise ImportError("No module named 'torch'")
        monkeypatch.setattr(build, "build_binding", no_torch)
    else:
        pytest.importorskip("torch")
        monkeypatch.setenv("CXX", "false" if broken == "compiler" else str(tmp_path / "nowhere"))
    assert build.build() == str(tmp_path / "libswconv.so")
    assert not stale.exists() and not os.path.exists(tmp_path / "_build")
    assert "native binding not built" in capsys.readouterr().err
