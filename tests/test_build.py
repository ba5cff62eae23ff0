"""The build's choice of tools (CPU): what is missing is named before anything is compiled."""
import pytest

from paper_2406_02701_amd import build as b


def test_missing_linker_is_named(monkeypatch):
    monkeypatch.setattr(b, "_compile", lambda src: pytest.fail("compiled without a linker"))
    monkeypatch.setenv("LD_LLD", "/nonexistent/ld.lld")
    with pytest.raises(RuntimeError, match="linker not found: /nonexistent/ld.lld"):
        b.build()


def test_another_linker_takes_the_place_of_rocms(monkeypatch):
    monkeypatch.delenv("LD_LLD", raising=False)
    monkeypatch.setattr(b.shutil, "which", lambda name: "/usr/bin/ld" if name == "ld" else None)
    assert b._linker() == "ld"
