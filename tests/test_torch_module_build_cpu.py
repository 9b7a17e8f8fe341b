"""The extension module with the C++ host path is only good for the torch it was built with: another torch makes its
object stale, and a module that does not load (or was built for another torch) leaves every call to the Python host
path, with a warning, because the kernels' library does not depend on torch."""
import sys
import warnings

import pytest
import torch

import paper_2605_17923_amd as package
from paper_2605_17923_amd import build, functional, lnmod


def test_another_torch_makes_the_object_stale(monkeypatch, tmp_path):
    compiled = []

    class Done:
        returncode = 0

    def run(cmd, **kw):
        compiled.append(cmd)
        open(cmd[cmd.index("-o") + 1], "w").close()
        return Done

    monkeypatch.setattr(build, "BUILD_DIR", str(tmp_path))
    monkeypatch.setattr(build.subprocess, "run", run)
    build._compile_torch(False)
    build._compile_torch(False)
    assert len(compiled) == 1                          # up to date the second time
    monkeypatch.setattr(torch, "__version__", "0.0.1+other")
    build._compile_torch(False)
    assert len(compiled) == 2
    build._compile_torch(False)
    assert len(compiled) == 2


@pytest.mark.parametrize("how", ["does not load", "another torch"])
def test_calls_take_the_python_path_where_the_module_is_unusable(monkeypatch, how):
    monkeypatch.setattr(lnmod, "_native", None)
    if how == "does not load":
        monkeypatch.setitem(sys.modules, package.__name__ + "._lnmod_torch", None)
        monkeypatch.delattr(package, "_lnmod_torch", raising=False)
    else:
        monkeypatch.setattr(torch, "__version__", "0.0.1+other")
    x, mod = torch.zeros(2, 3, 8), torch.zeros(2, 8)
    with pytest.warns(RuntimeWarning, match="_lnmod_torch"):
        with pytest.raises(ValueError, match="GPU"):   # the Python path's own check, not an import error
            functional.ln_modulate(x, mod, mod)
    with warnings.catch_warnings():
        warnings.simplefilter("error")                 # said once
        assert lnmod.native() is None
