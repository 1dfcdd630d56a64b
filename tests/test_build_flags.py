"""The build goes on without an option of the compiler's back end that the compiler does not have, and stops at anything else."""
import os
import shutil

import pytest

from paper_2605_15422_amd import build as B

pytestmark = pytest.mark.skipif(shutil.which(B._hipcc()) is None, reason="no hipcc")


def _build(tmp_path, monkeypatch, text, flags):
    (tmp_path / "one.hip").write_text(text)
    monkeypatch.setattr(B, "HERE", str(tmp_path))
    monkeypatch.setattr(B, "CSRC", str(tmp_path))
    monkeypatch.setattr(B, "LIB", str(tmp_path / "libone.so"))
    monkeypatch.setattr(B, "SOURCES", ["one.hip"])
    monkeypatch.setattr(B, "FILE_FLAGS", {"one.hip": flags})
    return B.build(verbose=False)


def test_unknown_back_end_option(tmp_path, monkeypatch):
    assert os.path.exists(_build(tmp_path, monkeypatch, "extern \"C\" int one() { return 1; }\n", ["-mllvm", "-no-such-option-of-the-allocator=1"]))


def test_an_error_in_the_source_still_stops_the_build(tmp_path, monkeypatch):
    with pytest.raises(RuntimeError, match="one.hip"):
        _build(tmp_path, monkeypatch, "int one() { return missing; }\n", ["-mllvm", "-no-such-option-of-the-allocator=1"])
