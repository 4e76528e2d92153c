"""dta_torch.so beside libdta.so (CPU): rebuilt by itself when it is missing or was made for another torch, and
done without, with a warning, where it cannot be used."""
import os
import sys
import types
import warnings

import pytest

import paper_2602_00482_amd as dta
from paper_2602_00482_amd import binding, build


def _call():
    import torch
    tree, p = dta.tree_build([-1, 0], [3, 4]), dta.AttnParams(2, 1, 64, 1.0, dta.F32)
    with pytest.raises(ValueError, match="q must be a contiguous CUDA tensor"):   # said by the general path
        dta.tree_attn_fwd(tree, p, torch.zeros(7, 2, 64), torch.zeros(7, 1, 64), torch.zeros(7, 1, 64))
    tree.destroy()


@pytest.mark.parametrize("module", [None, types.SimpleNamespace(), types.SimpleNamespace(built_for="torch 1.0, Python 2.7")])
def test_without_usable_compiled_calls_the_wrappers_make_them(monkeypatch, module):
    monkeypatch.setattr(binding, "_torch_calls", None)
    monkeypatch.setitem(sys.modules, "paper_2602_00482_amd.dta_torch", module)   # None: the import fails
    monkeypatch.setattr(dta, "dta_torch", module, raising=False)
    if module is None:
        monkeypatch.delattr(dta, "dta_torch")
    with pytest.warns(RuntimeWarning, match="dta_torch.so cannot be used"):
        _call()
    assert binding._torch_calls is False
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        _call()   # one warning


def test_the_built_module_is_the_one_of_this_torch():
    assert binding._calls().built_for == build.torch_stamp()
    assert not build._torch_stale()


@pytest.mark.parametrize("what", ["missing", "another torch", "older"])
def test_the_compiled_calls_are_rebuilt_by_themselves(monkeypatch, tmp_path, what):
    path = tmp_path / "dta_torch.so"
    if what != "missing":
        path.write_bytes(b"..." + (b"torch 1.0" if what == "another torch" else build.torch_stamp().encode()))
    if what == "older":
        os.utime(path, (1, 1))
    built = []
    monkeypatch.setattr(build, "TORCH_PATH", str(path))
    monkeypatch.setattr(build, "_stale", lambda: False)
    monkeypatch.setattr(build, "build", lambda: pytest.fail("built everything"))
    monkeypatch.setattr(build, "build_torch", lambda: built.append(1))
    build.ensure_built()
    assert built == [1]
    monkeypatch.setattr(build, "_cxx", lambda: None)   # no compiler: what is there is used
    assert build.ensure_built() == build.LIB_PATH and built == [1]
