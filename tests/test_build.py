"""What the build of the extension module (the per-step calls without ctypes) depends on; nothing is compiled here but
that module, into a temporary directory."""
import os
import subprocess
import sys

import pytest

from paper_2508_07014_amd import build


@pytest.fixture
def elsewhere(tmp_path, monkeypatch):
    """A library that is there and newer than its sources, and a place for the module."""
    lib, mod = tmp_path / "libpb.so", tmp_path / os.path.basename(build.CALL_LIB)
    lib.write_bytes(b"")
    monkeypatch.setattr(build, "LIB", str(lib))
    monkeypatch.setattr(build, "CALL_LIB", str(mod))
    return lib, mod


@pytest.mark.skipif(build.calls_compiler() is None, reason="no host compiler or Python headers")
def test_module_is_built_where_only_it_is_missing(elsewhere):
    lib, mod = elsewhere
    assert build.stale()
    assert build.build(force=False, out=str(lib)) == str(lib)
    assert mod.exists() and lib.read_bytes() == b""
    assert not build.stale()
    code = "import importlib.util as u, sys; s = u.spec_from_file_location('_pbcall', sys.argv[1]); m = u.module_from_spec(s); print(m.bind)"
    assert subprocess.run([sys.executable, "-c", code, str(mod)], capture_output=True).returncode == 0


@pytest.mark.skipif(build.calls_compiler() is None, reason="no host compiler or Python headers")
def test_module_older_than_its_source_is_stale(elsewhere):
    lib, mod = elsewhere
    mod.write_bytes(b"")
    assert not build.stale()
    src = os.path.getmtime(build.CALL_SOURCES[0])
    os.utime(mod, (src - 10, src - 10))
    assert build.stale()


def test_without_a_host_compiler_the_library_still_builds(elsewhere, monkeypatch, capsys):
    lib, mod = elsewhere
    monkeypatch.setattr(build.shutil, "which", lambda name: None)
    assert build.build(force=False, out=str(lib)) == str(lib)
    assert not mod.exists() and "ctypes" in capsys.readouterr().err
    assert not build.stale()       # (what cannot be built is not missed)
