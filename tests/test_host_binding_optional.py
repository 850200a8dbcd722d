"""The native marshalling extension (_prhs_host) is optional: without it, or
with one built for another torch or library version, the library loads and the
binding makes its calls through ctypes; without what its build needs, libprhs
is built alone."""

import sys
import types
import warnings

import pytest

from paper_2602_08329_amd import binding as B
from paper_2602_08329_amd import build

NAME = "paper_2602_08329_amd._prhs_host"


def reload(monkeypatch, module):
    """lib() as a process's first call finds it, with `module` in place of the
    extension (None: its import fails)."""
    monkeypatch.setitem(sys.modules, NAME, module)
    monkeypatch.delattr(sys.modules["paper_2602_08329_amd"], "_prhs_host", raising=False)
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_host", None)
    return B.lib()


def other(**attributes):
    m = types.ModuleType(NAME)
    m.bind = lambda *a: None
    m.schedule = lambda *a: pytest.fail("an extension that does not fit was called")
    for k, v in attributes.items():
        setattr(m, k, v)
    return m


@pytest.mark.parametrize("how", ["missing", "unmarked", "torch", "library"])
def test_library_loads_without_a_fitting_extension(monkeypatch, how):
    abi = B.lib().prhs_abi_version()
    module = {"missing": None, "unmarked": other(),
              "torch": other(torch_version="0.0.0", abi_version=abi),
              "library": other(torch_version=str(B.torch.__version__), abi_version=abi + 1)}[how]
    with pytest.warns(RuntimeWarning, match="_prhs_host"):
        reload(monkeypatch, module)
    assert B._host is None
    p = B.params(k=8, refresh_every=4, layer_group=2)
    assert [B.prhs_schedule(j, l, p) for j in (0, 1, 4) for l in (0, 1)] == [1, 0, 0, 0, 1, 0]
    assert B.prhs_max_topk(p, 100) == 8


def test_built_extension_is_taken(monkeypatch):
    h = pytest.importorskip(NAME)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        reload(monkeypatch, h)
    assert B._host is h


def test_build_leaves_the_extension_out_without_its_tools(monkeypatch, capsys):
    assert build.host_command("x.so") is not None
    monkeypatch.setattr(build.shutil, "which", lambda name: None)
    assert build.host_command("x.so") is None
    assert "g++" in capsys.readouterr().err
    monkeypatch.undo()
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": "/nonexistent"})
    assert build.host_command("x.so") is None
    assert "Python.h" in capsys.readouterr().err
