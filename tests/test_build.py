"""The build's own handling of compiler options (no device needed)."""
import os
import shutil

import pytest

from paper_2406_11836_amd import build


@pytest.mark.skipif(not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)), reason="no compiler")
def test_an_option_that_the_compiler_refuses(monkeypatch, tmp_path, capsys):
    src = tmp_path / "x.hip"
    src.write_text("extern \"C\" int answer() { return 42; }\n")
    monkeypatch.setattr(build, "BUILD_DIR", str(tmp_path))
    monkeypatch.setattr(build, "EXTRA", {"x.hip": ["-mllvm", "-no-such-option-of-this-compiler"]})
    assert os.path.exists(build._compile(str(src)))
    assert "no-such-option" in capsys.readouterr().err
    src.write_text("not a program\n")
    with pytest.raises(RuntimeError):
        build._compile(str(src))
