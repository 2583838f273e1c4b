"""What build() makes again, without compiling anything."""
import os

import pytest

from paper_2602_10016_amd import build


@pytest.fixture
def made(tmp_path, monkeypatch):
    for name in ("LIB", "TORCH_CALL", "MADE_FOR"):
        monkeypatch.setattr(build, name, str(tmp_path / name))
    done = []

    def make(name):
        done.append(name)
        open(getattr(build, name), "w").close()

    monkeypatch.setattr(build, "_build_library", lambda *args: make("LIB"))
    monkeypatch.setattr(build, "_build_torch_call", lambda: make("TORCH_CALL"))
    return done


def test_a_changed_torch_makes_the_module_again(made, monkeypatch):
    for expected in (["LIB", "TORCH_CALL"], []):
        made.clear()
        assert build.build() == build.LIB and made == expected
    monkeypatch.setattr(build, "_installed", lambda: "another torch")
    build.build()
    assert made == ["TORCH_CALL"]
    made.clear()
    build.build()
    assert made == []
    os.remove(build.MADE_FOR)  # built before this was noted
    build.build()
    assert made == ["TORCH_CALL"]


def test_sources_that_are_newer_and_force_make_both(made, monkeypatch):
    build.build()
    made.clear()
    build.build(force=True)
    assert made == ["LIB", "TORCH_CALL"]
    made.clear()
    monkeypatch.setattr(build, "_deps_mtime", lambda: os.path.getmtime(build.LIB) + 1)
    build.build()
    assert made == ["LIB", "TORCH_CALL"]
