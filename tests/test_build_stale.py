"""What a build of stale files only compiles again (CPU only; a stand-in for the compiler that writes empty objects)."""
import os
import stat

import pytest

from paper_2307_14995_amd import build


def test_objects_of_other_flags_are_compiled_again(monkeypatch, tmp_path):
    hipcc, log = tmp_path / "hipcc", tmp_path / "log"
    hipcc.write_text(f'#!/bin/sh\necho "$*" >> {log}\nwhile [ "$1" != -o ]; do shift; done\n: > "$2"\n')
    hipcc.chmod(hipcc.stat().st_mode | stat.S_IXUSR)
    monkeypatch.setenv("HIPCC", str(hipcc))
    for name in ("OBJ", "SAN_OBJ"):
        monkeypatch.setattr(build, name, str(tmp_path / name))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setattr(build, "SAN_LIB", str(tmp_path / "san.so"))
    monkeypatch.setattr(build, "marshalling_is_stale", lambda: False)
    os.makedirs(build.SAN_OBJ)

    def commands(make):
        log.write_text("")
        make()
        return log.read_text().splitlines()

    def stale_only():
        build.build_library(force=False, marshalling=False)

    every = len(build.sources()) + 1                      # and the link
    for make, is_stale in ((stale_only, build.is_stale), (build.build_sanitized, None)):
        assert len(commands(make)) == every
        assert commands(make) == [] and not (is_stale and is_stale())
    monkeypatch.setattr(build, "HIPCC_FLAGS", build.HIPCC_FLAGS + ["-DOTHER"])
    for make, is_stale in ((stale_only, build.is_stale), (build.build_sanitized, None)):
        assert not is_stale or is_stale()
        again = commands(make)
        assert len(again) == every and all("-DOTHER" in c for c in again[:-1])
        assert commands(make) == []
    # a compilation that failed is not taken for done
    hipcc.write_text("#!/bin/sh\nexit 1\n")
    monkeypatch.setattr(build, "HIPCC_FLAGS", build.HIPCC_FLAGS[:-1])
    with pytest.raises(RuntimeError):
        stale_only()
    assert build.is_stale()
