"""The build on the host: the C library does not depend on the Python call
module, and the compiler may be given as a path, a link or a name on PATH."""

import os
import stat

import pytest

from paper_2609_33269_amd import build


def _fake_rocm(root):
    """A ROCm tree whose hipcc writes its -o file."""
    (root / "bin").mkdir(parents=True)
    (root / "include" / "hip").mkdir(parents=True)
    (root / "include" / "hip" / "hip_runtime.h").write_text("")
    hipcc = root / "bin" / "hipcc"
    hipcc.write_text('#!/bin/sh\nwhile [ "$1" != -o ]; do shift; done\necho built > "$2"\n')
    hipcc.chmod(hipcc.stat().st_mode | stat.S_IXUSR)
    return hipcc


def test_library_is_linked_when_the_call_module_fails(tmp_path, monkeypatch):
    monkeypatch.setattr(build, "HIPCC", str(_fake_rocm(tmp_path / "rocm")))
    monkeypatch.setattr(build, "BUILD_DIR", str(tmp_path / "obj"))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libqwam.so"))

    def no_headers(verbose):
        raise RuntimeError("no PyTorch headers")

    monkeypatch.setattr(build, "_build_call_module", no_headers)
    with pytest.raises(RuntimeError, match="no PyTorch headers"):
        build.build()
    assert os.path.exists(tmp_path / "libqwam.so")


@pytest.mark.parametrize("how", ["path", "name", "link"])
def test_rocm_root(tmp_path, monkeypatch, how):
    hipcc = _fake_rocm(tmp_path / "rocm")
    if how == "path":
        given = str(hipcc)
    elif how == "name":
        monkeypatch.setenv("PATH", str(hipcc.parent), prepend=os.pathsep)
        given = "hipcc"
    else:
        (tmp_path / "elsewhere" / "bin").mkdir(parents=True)
        given = str(tmp_path / "elsewhere" / "bin" / "hipcc")
        os.symlink(hipcc, given)
    monkeypatch.setattr(build, "HIPCC", given)
    assert build._rocm_root() == str(tmp_path / "rocm")
