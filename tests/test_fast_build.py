"""The binding's native calls are an addition: where they cannot be built or loaded, the library loads and its calls go through
ctypes as if they were not there."""
import os
import stat

import pytest

from paper_1802_04730_amd import build as tcbuild, tc355


def script(path, text):
    path.write_text("#!/bin/sh\n" + text)
    path.chmod(path.stat().st_mode | stat.S_IXUSR)
    return str(path)


@pytest.fixture
def fresh(tmp_path, monkeypatch):
    """The binding as before its first call, its native calls not yet built (in a folder of this test)."""
    if not os.path.exists(tcbuild.LIB):
        tcbuild.build(force=True)
    monkeypatch.setattr(tc355, "_LIB", None)
    monkeypatch.setattr(tc355, "_FAST", None)
    monkeypatch.setattr(tcbuild, "FAST", str(tmp_path / "_fast.so"))
    monkeypatch.setattr(tcbuild, "FAST_STAMP", str(tmp_path / "_fast.so.srchash"))
    return tmp_path


def check_general_path():
    assert tc355._FAST is None and tc355.tc355_version() >= 100
    assert tc355.tc_sconv2d_infer(9, 8, 3, 3, 2, 1) == (4, 6)
    with pytest.raises((TypeError, ValueError, AttributeError)):
        tc355.tc_tbmm(None, None, None)


def test_no_compiler(fresh, monkeypatch):
    monkeypatch.setenv("CXX", str(fresh / "nothing"))
    check_general_path()


def test_compiler_without_headers(fresh, monkeypatch):
    monkeypatch.setenv("CXX", script(fresh / "cxx", "echo Python.h: no such file >&2\nexit 1\n"))
    with pytest.warns(RuntimeWarning, match="Python.h: no such file"):
        tc355.lib()
    check_general_path()


def test_folder_that_cannot_be_written(fresh, monkeypatch):
    monkeypatch.setattr(tcbuild, "FAST", str(fresh / "missing" / "_fast.so"))
    monkeypatch.setattr(tcbuild, "FAST_STAMP", str(fresh / "missing" / "_fast.so.srchash"))
    monkeypatch.setenv("CXX", script(fresh / "cxx", "exit 0\n"))  # (quick: the stamp is what fails)
    with pytest.warns(RuntimeWarning):
        tc355.lib()
    check_general_path()


def test_module_that_cannot_be_loaded(fresh):
    (fresh / "_fast.so").write_bytes(b"not a module")
    (fresh / "_fast.so.srchash").write_text(tcbuild.fast_hash() + "\n")
    with pytest.warns(RuntimeWarning):
        tc355.lib()
    check_general_path()


def test_the_library_is_built_without_them(fresh, monkeypatch):
    monkeypatch.setattr(tcbuild, "LIB", str(fresh / "lib.so"))
    monkeypatch.setattr(tcbuild, "STAMP", str(fresh / "lib.so.srchash"))
    monkeypatch.setenv("HIPCC", script(fresh / "hipcc", 'while [ "$1" != -o ]; do shift; done\necho built > "$2"\n'))
    monkeypatch.setenv("CXX", str(fresh / "nothing"))
    with pytest.warns(RuntimeWarning, match="_fast.so"):
        assert tcbuild.build(force=True) == str(fresh / "lib.so")
    assert (fresh / "lib.so").read_text() == "built\n" and not tcbuild.is_stale() and tcbuild.fast_is_stale()


def test_a_module_is_written_as_a_whole(fresh, monkeypatch):
    """What another process may be loading is replaced, never written into; a compiler that fails half-way leaves it alone."""
    out = fresh / "_fast.so"
    out.write_text("the one before")
    to_output = 'while [ "$1" != -o ]; do shift; done\necho half > "$2"\n'
    monkeypatch.setenv("CXX", script(fresh / "cxx", to_output + "exit 1\n"))
    with pytest.raises(RuntimeError):
        tcbuild.build_fast()
    assert out.read_text() == "the one before" and tcbuild.fast_is_stale()
    monkeypatch.setenv("CXX", script(fresh / "cxx", to_output + 'echo whole > "$2"\n'))
    with open(out) as before:
        tcbuild.build_fast()
        assert before.read() == "the one before"
    assert out.read_text() == "whole\n" and not tcbuild.fast_is_stale()
    assert sorted(p.name for p in fresh.iterdir()) == ["_fast.so", "_fast.so.srchash", "cxx"]


def test_a_stamp_names_what_the_compiler_read(fresh, monkeypatch):
    """Other flags, or a source that is edited while it compiles, leave the module stale."""
    source = fresh / "fast_call.cpp"
    source.write_text("// one\n")
    monkeypatch.setattr(tcbuild, "FAST_SOURCE", str(source))
    compiler = 'while [ "$1" != -o ]; do shift; done\necho module > "$2"\n'
    monkeypatch.setenv("CXX", script(fresh / "cxx", compiler + "echo // two > %s\n" % source))
    tcbuild.build_fast()
    assert tcbuild.fast_is_stale()
    monkeypatch.setenv("CXX", script(fresh / "cxx", compiler))
    tcbuild.build_fast()
    assert not tcbuild.fast_is_stale()
    monkeypatch.setattr(tcbuild, "FAST_FLAGS", tcbuild.FAST_FLAGS + ["-g"])
    assert tcbuild.fast_is_stale()
