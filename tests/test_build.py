"""What a build needs: the library hipcc alone, the native part of the binding a C++ compiler and torch's headers."""
import os
import stat

import pytest

from paper_2603_27462_amd import build


def _paths(tmp_path, monkeypatch):
    hipcc = tmp_path / "hipcc"      # writes something to the file behind -o
    hipcc.write_text('#!/bin/sh\nwhile [ $# -gt 1 ]; do [ "$1" = -o ] && echo built > "$2"; shift; done\n')
    hipcc.chmod(hipcc.stat().st_mode | stat.S_IXUSR)
    monkeypatch.setenv("HIPCC", str(hipcc))
    monkeypatch.setattr(build, "LIB_PATH", str(tmp_path / "librsr.so"))
    monkeypatch.setattr(build, "CALL_PATH", str(tmp_path / "_rsr_call.so"))


@pytest.mark.parametrize("compiler", ["/nonexistent/g++", "/bin/false"])
def test_library_without_the_native_part(tmp_path, monkeypatch, compiler):
    _paths(tmp_path, monkeypatch)
    monkeypatch.setenv("CXX", compiler)
    with open(build.CALL_PATH, "w") as f:
        f.write("of an earlier build")
    with pytest.warns(UserWarning, match="native part"):
        assert build.build_library() == build.LIB_PATH
    assert os.path.exists(build.LIB_PATH) and not os.path.exists(build.CALL_PATH)
    assert sorted(os.listdir(tmp_path)) == ["hipcc", "librsr.so"]       # no temporary files either
