"""What build.py makes where parts of its surroundings are missing (stand-ins for the compilers, nothing is compiled)."""
import os
import stat
import sys

import pytest

from paper_2009_06693_amd import build


@pytest.fixture
def tools(tmp_path, monkeypatch):
    """A hipcc and a clang++ beside it that write what they are asked for; the folder is all there is on PATH."""
    for name in ("hipcc", "amdclang++"):
        exe = tmp_path / name
        exe.write_text(f"#!{sys.executable}\nimport sys\n"
                       f"open(sys.argv[sys.argv.index('-o') + 1], 'w').write({name!r})\n")
        exe.chmod(exe.stat().st_mode | stat.S_IXUSR)
    monkeypatch.setenv("PATH", str(tmp_path))
    monkeypatch.delenv("CXX", raising=False)
    for name, path in (("HIPCC", "hipcc"), ("LIB", "libnd.so"), ("CALL_LIB", "_nd_call.so"), ("OBJ", "obj")):
        monkeypatch.setattr(build, name, str(tmp_path / path))
    return tmp_path


def test_the_library_is_linked_without_torch(tools, monkeypatch, capsys):
    monkeypatch.setitem(sys.modules, "torch", None)  # importing it raises, as where it is not installed
    monkeypatch.setattr("importlib.util.find_spec", lambda name, package=None: None)
    assert build.build() == build.LIB
    assert os.path.exists(build.LIB) and not os.path.exists(build.CALL_LIB)
    assert "torch is not installed" in capsys.readouterr().err


def test_the_library_is_linked_where_the_binding_does_not_compile(tools, monkeypatch):
    monkeypatch.setenv("CXX", str(tools / "missing"))
    with pytest.raises(FileNotFoundError):
        build.build()
    assert os.path.exists(build.LIB)


def test_the_binding_is_compiled_without_gcc(tools):
    build.build()
    assert open(build.CALL_LIB).read() == "amdclang++"
