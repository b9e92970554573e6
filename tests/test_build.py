"""The order of the build and the loading of the optional call module (nothing is compiled here)."""
import subprocess
import warnings

import pytest

from paper_2512_23367_amd import binding as ql
from paper_2512_23367_amd import build


def test_libraries_are_built_where_the_call_module_cannot_be(tmp_path, monkeypatch, capsys):
    """No host compiler, Python.h or torch headers: the libraries depend on none of them."""
    linked, stale = [], tmp_path / "_qlcall.so"
    stale.write_bytes(b"of an earlier build")

    def fails():
        raise subprocess.CalledProcessError(1, ["g++"])

    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    monkeypatch.setattr(build, "CALL_MODULE", str(stale))
    monkeypatch.setattr(build, "_compile", lambda src: src + ".o")
    monkeypatch.setattr(build, "_link", lambda objs, lib: linked.append(lib))
    monkeypatch.setattr(build, "_build_call_module", fails)
    assert build.build() == build.LIB and linked == [build.LIB, build.PROBE_LIB]
    assert "_qlcall" in capsys.readouterr().err and not stale.exists()      # said, and no module of other sources is left


def test_a_library_that_does_not_compile_is_an_error(tmp_path, monkeypatch):
    def fails(src):
        raise subprocess.CalledProcessError(1, ["hipcc"])

    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    monkeypatch.setattr(build, "_compile", fails)
    monkeypatch.setattr(build, "_build_call_module", lambda: None)
    with pytest.raises(subprocess.CalledProcessError):
        build.build()


@pytest.mark.parametrize("error,warns", [(ModuleNotFoundError("No module named '_qlcall'"), False), (ImportError("undefined symbol: _ZN3c10"), True)])
def test_a_call_module_that_does_not_load_is_reported_and_a_missing_one_is_not(error, warns, monkeypatch):
    def fails(name):
        raise error

    lib = ql.lib()
    monkeypatch.setattr(ql, "_native", None)
    monkeypatch.setattr(ql, "import_module", fails)
    with warnings.catch_warnings(record=True) as caught:
        warnings.simplefilter("always")
        ql._bind_native(lib)
    assert ql._native is None and [("undefined symbol" in str(w.message)) for w in caught] == [True] * warns
