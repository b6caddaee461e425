"""The C library builds without the Python entry points; each has a stamp that covers what it is built from."""
import subprocess

import pytest

from paper_2505_11432_amd import build


def test_library_needs_no_torch_and_no_host_compiler(tmp_path, monkeypatch):
    monkeypatch.setattr(build, "OBJ_DIR", str(tmp_path))
    for name in ("LIB_PATH", "CEILINGS_LIB_PATH", "NATIVE_PATH", "STAMP_PATH", "NATIVE_STAMP_PATH"):
        monkeypatch.setattr(build, name, str(tmp_path / name))
    monkeypatch.setattr(build, "_compile", lambda src: src)

    def no_torch(name):
        raise build.metadata.PackageNotFoundError(name)

    def run(cmd, **kw):
        if cmd[0] != build.HIPCC:
            return subprocess.CompletedProcess(cmd, 1, "", "no host compiler")
        (tmp_path / cmd[cmd.index("-o") + 1]).touch()
        return subprocess.CompletedProcess(cmd, 0, "", "")

    monkeypatch.setattr(build.metadata, "version", no_torch)
    monkeypatch.setattr(build.subprocess, "run", run)
    build.build(verbose=False, native=False)
    assert build.is_current() and not build.native_is_current()
    with pytest.raises(RuntimeError, match="no host compiler"):
        build.build(verbose=False)
    assert build.is_current() and not build.native_is_current()      # the library stays usable


def test_module_of_another_interpreter_or_toolchain_is_stale(monkeypatch):
    build.ensure_built()
    assert build.is_current() and build.native_is_current()
    for obj, name, value in ((build.sysconfig, "get_config_var", lambda key: ".cpython-399-x86_64-linux-gnu.so"),
                             (build, "CXX", "another-g++"), (build, "NATIVE_CFLAGS", build.NATIVE_CFLAGS + ["-DX"]),
                             (build, "NATIVE_LIBS", build.NATIVE_LIBS[1:]), (build.metadata, "version", lambda name: "0.0")):
        with monkeypatch.context() as m:
            m.setattr(obj, name, value)
            assert build.is_current() and not build.native_is_current()
