"""Which marshalling module the binding uses, without a GPU: the one that is there, if it is for this interpreter and torch."""
import os
import subprocess
import sys
import types
import warnings

import pytest

from paper_2109_09868_amd import binding, build


@pytest.fixture
def fresh(monkeypatch):
    import paper_2109_09868_amd as package
    monkeypatch.setattr(binding, "_ordinary", None)
    monkeypatch.delattr(package, "_marshal", raising=False)
    monkeypatch.delitem(sys.modules, "paper_2109_09868_amd._marshal", raising=False)
    monkeypatch.setattr(binding, "load", lambda lib=object(): lib)
    return monkeypatch


def test_no_module_means_ctypes_without_a_word(fresh, tmp_path):
    fresh.setattr(binding, "MARSHAL_PATH", str(tmp_path / "_marshal.so"))
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        assert binding._marshal() == (None, None)


@pytest.mark.parametrize("module", [None, types.SimpleNamespace(), types.SimpleNamespace(built_for="cpython-39 torch 1.0")],
                         ids=["cannot be loaded", "does not say", "for another torch"])
def test_a_module_that_does_not_fit_is_not_used_and_says_so(fresh, tmp_path, module):
    (tmp_path / "_marshal.so").write_bytes(b"")
    fresh.setattr(binding, "MARSHAL_PATH", str(tmp_path / "_marshal.so"))
    fresh.setitem(sys.modules, "paper_2109_09868_amd._marshal", module)          # None: the import fails
    with pytest.warns(RuntimeWarning, match="build it again"):
        assert binding._marshal() == (None, None)
    with warnings.catch_warnings():                                              # once, not at every call
        warnings.simplefilter("error")
        assert binding._marshal() == (None, None)


def test_the_module_is_built_without_gcc_too(monkeypatch, tmp_path):
    which = build.shutil.which
    monkeypatch.setattr(build.shutil, "which", lambda name: None if name == "g++" else which(name))
    out = build.build_marshal(out=str(tmp_path / "_marshal.so"))
    program = ("import torch, importlib.machinery as m, importlib.util as u; s = u.spec_from_file_location('_marshal', %r); "
               "x = u.module_from_spec(s); s.loader.exec_module(x); print(x.built_for)" % out)
    r = subprocess.run([sys.executable, "-c", program], capture_output=True, text=True, cwd=os.path.dirname(build.PKG_DIR))
    assert r.stdout.strip() == binding.marshal_target(), r.stderr
