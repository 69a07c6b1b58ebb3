"""The build's bookkeeping (CPU only): the linker that joins the objects of the
level passes comes from the compiler in use, and objects left by an earlier
build are told from those of the present sources."""

import os

import pytest

from paper_2602_01888_amd import build


def test_linker_is_the_compilers(monkeypatch, tmp_path):
    hipcc = tmp_path / "hipcc"
    hipcc.write_text('#!/bin/sh\n[ "$1" = -print-prog-name=ld.lld ] && echo /elsewhere/ld.lld\n')
    hipcc.chmod(0o755)
    monkeypatch.setattr(build, "HIPCC", str(hipcc))
    assert build.linker() == "/elsewhere/ld.lld"


@pytest.fixture
def tree(monkeypatch, tmp_path):
    """A copy of the build's layout, every object a second newer than its sources."""
    csrc, objs = tmp_path / "csrc", tmp_path / "_build"
    csrc.mkdir()
    objs.mkdir()
    monkeypatch.setattr(build, "CSRC", str(csrc))
    monkeypatch.setattr(build, "OBJDIR", str(objs))
    header = csrc / "tomg_internal.h"
    monkeypatch.setattr(build, "HEADERS", [str(header)])

    def put(path, t):
        open(path, "w").close()
        os.utime(path, (t, t))
    for s in build.SOURCES:
        put(str(csrc / s), 1000)
        put(build.object_of(s), 1001)
    put(str(header), 1000)
    put(str(objs / "fused.hip.o"), 1002)
    return put


def test_present_objects_are_current(tree):
    assert not build.stale_objects()


@pytest.mark.parametrize("name", build.SOURCES + ["tomg_internal.h"])
def test_edited_source_makes_objects_stale(tree, name):
    tree(os.path.join(build.CSRC, name), 1003)
    assert build.stale_objects()


@pytest.mark.parametrize("name", ["api.hip.o", "fused.hip.o", "fused.hip.part.o",
                                  "tile.hip.part.o", "march.hip.part.o", "tail.hip.o"])
def test_missing_object_is_stale(tree, name):
    os.remove(os.path.join(build.OBJDIR, name))
    assert build.stale_objects()


def test_join_older_than_its_parts_is_stale(tree):
    tree(build.object_of("tile.hip"), 1004)
    assert build.stale_objects()
