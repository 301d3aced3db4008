"""The order of a build: the library does not wait for the binding's C++ half, which needs torch's headers."""
import os
import stat

import pytest

from paper_2409_18747_amd import build


@pytest.fixture
def sandbox(tmp_path, monkeypatch):
    """A compiler that writes down what it is asked and makes the file, in the place of hipcc."""
    hipcc = tmp_path / "rocm" / "bin" / "hipcc"
    hipcc.parent.mkdir(parents=True)
    hipcc.write_text('#!/bin/sh\nwhile [ $# -gt 0 ]; do [ "$1" = -o ] && echo made > "$2"; shift; done\n')
    hipcc.chmod(hipcc.stat().st_mode | stat.S_IXUSR)
    monkeypatch.setattr(build, "HIPCC", str(hipcc))
    for name, path in (("LIB", "libcottn.so"), ("MARSHAL", "_marshal.so"), ("OBJ_DIR", "objects")):
        monkeypatch.setattr(build, name, str(tmp_path / path))
    return tmp_path


def test_library_is_linked_where_the_binding_does_not_compile(sandbox, monkeypatch):
    monkeypatch.setenv("CXX", "false")
    with pytest.raises(RuntimeError, match=r"marshal\.cpp"):
        build.build()
    assert os.path.exists(build.LIB) and not os.path.exists(build.MARSHAL)


def test_library_is_linked_without_torch(sandbox, monkeypatch):
    monkeypatch.setitem(__import__("sys").modules, "torch", None)   # `import torch` raises
    with pytest.raises(ImportError):
        build.build()
    assert os.path.exists(build.LIB) and not os.path.exists(build.MARSHAL)


def test_headers_of_the_compilers_own_rocm(sandbox, monkeypatch):
    cxx = sandbox / "cxx"
    cxx.write_text('#!/bin/sh\necho "$@" > %s/asked\n%s "$@"\n' % (sandbox, build.HIPCC))
    cxx.chmod(cxx.stat().st_mode | stat.S_IXUSR)
    monkeypatch.setenv("CXX", str(cxx))
    build.build()
    assert os.path.exists(build.LIB) and os.path.exists(build.MARSHAL)
    assert "-isystem %s/rocm/include" % sandbox in (sandbox / "asked").read_text()
