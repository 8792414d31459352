"""Opening the library where its native marshalling cannot be had: no compiler, a file that is none, one built
for something else.  Every call is then marshalled in Python, with a warning; nothing else is lost."""
import os
import stat

import pytest
import torch

import paper_2307_14995_amd as ltn
from paper_2307_14995_amd import binding, build


@pytest.fixture
def fresh(monkeypatch, tmp_path):
    """As in a process that has not opened the library yet, its marshalling at a place of its own."""
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_native", None)
    path = str(tmp_path / "_ltn_torch.so")
    monkeypatch.setattr(build, "TORCH_LIB", path)
    yield path
    monkeypatch.undo()
    binding._bind_native(binding.load_library())         # (the module's functions are one set a process)


def opens_without(path):
    with pytest.warns(RuntimeWarning, match="native marshalling"):
        assert ltn.ltn_attn_pick_block(128, torch.bfloat16) == 64
    assert binding._fast().fwd(1, 2, 3) is None
    with pytest.raises(ValueError, match="GPU"):
        ltn.ltn_gate_bwd(*(torch.zeros(2, 64) for _ in range(3)))


def compiler(path, script):
    path.write_text("#!/bin/sh\n" + script)
    path.chmod(path.stat().st_mode | stat.S_IXUSR)
    return str(path)


def test_no_compiler(fresh, monkeypatch):
    monkeypatch.setenv("CXX", "/nonexistent/c++")
    opens_without(fresh)


def test_compiler_without_torch_headers(fresh, monkeypatch, tmp_path):
    monkeypatch.setenv("CXX", compiler(tmp_path / "cxx", "echo no such header >&2; exit 1\n"))
    opens_without(fresh)


def test_a_file_that_is_no_extension(fresh):
    with open(fresh, "wb") as f:
        f.write(b"half a file")
    opens_without(fresh)
    assert build.marshalling_is_stale()


def test_built_for_another_torch_or_header(monkeypatch):
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_native", None)
    ltn.load_library()
    assert binding._native.built_for == build.marshalling_id() and not build.marshalling_is_stale()
    real = build.marshalling_id
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(build, "marshalling_id", lambda: real() + " other")
    assert build.marshalling_is_stale()
    opens_without(build.TORCH_LIB)


def test_a_failed_build_leaves_the_old_file(monkeypatch, tmp_path):
    path = str(tmp_path / "_ltn_torch.so")
    monkeypatch.setattr(build, "TORCH_LIB", path)
    with open(path, "w") as f:
        f.write("old")
    # writes half of its output, then fails
    monkeypatch.setenv("CXX", compiler(tmp_path / "cxx", 'while [ "$1" != -o ]; do shift; done; echo half > "$2"; exit 1\n'))
    with pytest.raises(RuntimeError, match="failed on"):
        build.build_marshalling()
    assert open(path).read() == "old" and sorted(os.listdir(tmp_path)) == ["_ltn_torch.so", "cxx"]


def test_the_library_is_complete_when_the_marshalling_fails(monkeypatch, tmp_path):
    # (nothing stale: the build of the library itself is nothing here)
    monkeypatch.setattr(build, "sources", lambda: [])
    monkeypatch.setattr(build, "_stale", lambda target, deps: target == build.LIB)
    monkeypatch.setattr(build, "marshalling_is_stale", lambda: True)
    linked = []

    class Result:
        returncode, stdout, stderr = 0, "", ""

    monkeypatch.setattr(build.subprocess, "run", lambda cmd, **k: linked.append(cmd) or Result())

    def fails(verbose):
        raise RuntimeError("no marshalling")

    monkeypatch.setattr(build, "build_marshalling", fails)
    with pytest.raises(RuntimeError, match="no marshalling"):
        build.build_library(force=False)
    assert len(linked) == 1 and linked[0][-1] == build.LIB
    build.build_library(force=False, marshalling=False)
    assert len(linked) == 2
