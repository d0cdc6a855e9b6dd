"""Build steps keep the compiler's output and name themselves when they fail."""
from __future__ import annotations

import os

import pytest

from paper_1704_04374_amd import build


def test_failed_step_says_what_failed(tmp_path, monkeypatch):
    monkeypatch.setattr(build, "BUILD", str(tmp_path))
    build.run_step("good", ["sh", "-c", "echo fine"])
    assert "fine" in (tmp_path / "good.log").read_text()
    with pytest.raises(RuntimeError, match=r"bad: exit status 3 after [\d.]+ s[\s\S]*sh -c[\s\S]*oops"):
        build.run_step("bad", ["sh", "-c", "echo oops >&2; exit 3"])
    assert "oops" in (tmp_path / "bad.log").read_text()
    with pytest.raises(RuntimeError, match="exit status -9"):    # ended by a signal
        build.run_step("killed", ["sh", "-c", "kill -9 $$"])


def test_every_source_is_built():
    """No kernel or host source is left out of both libraries."""
    built = set(build.SOURCES) | set(build.CONTRACT_SOURCES)
    there = {f for f in os.listdir(build.CSRC) if f.endswith((".hip", ".cpp"))}
    assert built == there
