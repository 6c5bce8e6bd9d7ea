"""The native gatherer of module descriptors is optional: without g++ or torch's
headers the library still builds, and without the module (or with one for another
torch) the binding's Python checks take every call."""
import os
import sys

import pytest
import torch

import paper_2606_11660_amd as P
from paper_2606_11660_amd import build as B


def test_it_is_built_here():
    from paper_2606_11660_amd import _marshal
    assert os.path.samefile(_marshal.__file__, B.MARSHAL)


@pytest.mark.parametrize("how", ["no g++", "compile error"])
def test_a_failed_build_leaves_no_stale_module(how, tmp_path, monkeypatch, capsys):
    so = tmp_path / "_marshal.so"
    so.write_bytes(b"stale")
    monkeypatch.setattr(B, "MARSHAL", str(so))
    if how == "no g++":
        monkeypatch.setattr(B.shutil, "which", lambda name: None)
    else:
        monkeypatch.setattr(B, "_marshal_command", lambda out: ["false"])
    assert B.build_marshal() is False
    assert not so.exists() and "was not built" in capsys.readouterr().err


def test_calls_run_the_python_checks_without_it(monkeypatch):
    monkeypatch.setattr(P, "_native_modules", None)
    monkeypatch.setitem(sys.modules, "paper_2606_11660_amd._marshal", None)  # the import fails
    a, g = torch.zeros((8, 64)), torch.zeros((8, 128))
    mod = P.Module(a, g, torch.zeros((128, 16)), torch.zeros((64, 16)), 0)
    out = torch.zeros((2, 256))
    with pytest.warns(RuntimeWarning, match="check their modules in Python"):
        with pytest.raises(ValueError, match="same GPU"):  # the last of the Python checks
            P.attr_project([mod], 16, 2, 4, out)
    with pytest.raises(ValueError, match="rows, the call writes"):
        P.attr_project([mod], 16, 3, 4, out)
