"""The build: the binding's native argument marshalling is an extra, without which the library is built all the same."""
import os
import sys
import sysconfig

import pytest

from paper_2605_23163_amd import build as b


@pytest.fixture
def out(monkeypatch, tmp_path):
    monkeypatch.setattr(b, "LIB", str(tmp_path / "libfdd.so"))
    monkeypatch.setattr(b, "MARSHAL", str(tmp_path / os.path.basename(b.MARSHAL)))
    return tmp_path


def without_hipcc(monkeypatch):
    """HIP compilations leave an empty file; other commands run"""
    run = b._run

    def fake(cmd):
        if cmd[0] == b.HIPCC:
            open(cmd[cmd.index("-o") + 1], "w").close()
        else:
            run(cmd)
    monkeypatch.setattr(b, "_run", fake)
    monkeypatch.setattr(b, "ROOT", os.path.dirname(b.LIB))


@pytest.mark.parametrize("cxx", ["/nowhere/g++", "false"])
def test_library_is_built_without_a_host_compiler(monkeypatch, out, capsys, cxx):
    if b.marshal_command("x") is None:
        pytest.skip("no torch headers here")
    stale = [out / "_marshal.so", out / os.path.basename(b.MARSHAL)]
    for f in stale:
        f.write_text("stale")
    monkeypatch.setenv("CXX", cxx)
    without_hipcc(monkeypatch)
    assert b.build() == b.LIB and os.path.exists(b.LIB)
    assert not any(f.exists() for f in stale) and not list(out.glob("*.tmp"))
    assert "marshalled in Python" in capsys.readouterr().out


def test_torch_without_headers(monkeypatch, tmp_path):
    (tmp_path / "torch").mkdir()
    (tmp_path / "torch" / "__init__.py").write_text("")
    monkeypatch.delitem(sys.modules, "torch", raising=False)
    monkeypatch.syspath_prepend(str(tmp_path))
    assert b.marshal_command("x") is None


def test_module_is_named_for_this_interpreter():
    assert os.path.basename(b.MARSHAL) == "_marshal" + sysconfig.get_config_var("EXT_SUFFIX")
