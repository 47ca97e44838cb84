"""The binding's native part is an accelerator: where it cannot be loaded, or was built for another torch, the
ctypes path takes every call.  (No GPU needed.)"""
import subprocess
import sys
import types

import pytest

import paper_2602_09323_amd as coopt
from paper_2602_09323_amd import binding

NAME = "paper_2602_09323_amd._binding"


@pytest.fixture()
def unbound(monkeypatch):
    coopt.load_library()
    monkeypatch.setattr(binding, "_native", None)
    monkeypatch.delattr(sys.modules["paper_2602_09323_amd"], "_binding", raising=False)


def _spec(module):
    # (where nothing is built there is no module to look for: the test brings its own)
    module.__spec__ = types.SimpleNamespace(name=NAME, loader=None, origin=None, parent="paper_2602_09323_amd")
    return module


@pytest.mark.parametrize("module", [types.ModuleType(NAME), types.ModuleType(NAME)], ids=["another torch", "before versions"])
def test_built_for_another_torch(unbound, monkeypatch, request, module):
    if "another" in request.node.callspec.id:
        module.built_for = "0.0.0"
    module.bind = lambda *a: pytest.fail("bound")
    monkeypatch.setitem(sys.modules, NAME, _spec(module))
    with pytest.warns(RuntimeWarning, match="native part is left out"):
        assert binding._fast() is None
    assert binding._native is False                     # once and for all: no second try, no second warning
    assert binding._fast() is None
    with pytest.raises(coopt.CooptError, match="required tensor is None"):
        coopt.paged_gqa_reduce(None, None, None, None, 16, 1, None, coopt.Shape(1, 1, 1, 64, 16, 1, 1, 0, 1.0))


def test_does_not_import(unbound, monkeypatch):
    class Finder:
        @staticmethod
        def find_spec(name, path=None, target=None):
            if name != NAME:
                return None
            from importlib.machinery import ModuleSpec

            class Loader:
                @staticmethod
                def create_module(spec):
                    raise ImportError("undefined symbol")

                @staticmethod
                def exec_module(module):
                    pass
            return ModuleSpec(name, Loader())
    monkeypatch.delitem(sys.modules, NAME, raising=False)
    monkeypatch.setattr(sys, "meta_path", [Finder] + sys.meta_path)
    with pytest.warns(RuntimeWarning, match="undefined symbol"):
        assert binding._fast() is None


def test_libraries_need_no_torch_headers(monkeypatch, tmp_path, capsys):
    """The C libraries are linked, and count as built, where the native part does not compile; another torch does not."""
    from paper_2602_09323_amd import build
    empty = tmp_path / "empty.cpp"
    empty.write_text("")

    def compiled(src):
        obj = str(tmp_path / (src + ".o"))
        subprocess.run(["g++", "-fPIC", "-c", str(empty), "-o", obj], check=True)
        return obj

    def fails():
        raise RuntimeError("no headers")
    for name in ("LIB", "PROBE_LIB", "BINDING", "BINDING_STAMP", "BUILD"):
        monkeypatch.setattr(build, name, str(tmp_path / name), raising=False)
    monkeypatch.setattr(build, "_compile", compiled)
    monkeypatch.setattr(build, "_build_binding", fails)
    (tmp_path / "BINDING").write_text("of older sources")
    assert build.build(force=True) == str(tmp_path / "LIB")
    assert (tmp_path / "LIB").exists() and (tmp_path / "PROBE_LIB").exists() and not (tmp_path / "BINDING").exists()
    assert "ctypes takes its calls: no headers" in capsys.readouterr().err
    assert not build.needs_build()
    monkeypatch.setattr(build, "_torch_version", lambda: "0.0.0")
    assert build.needs_build()
