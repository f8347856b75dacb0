"""The native half of the binding as far as it goes without a GPU: loading it, and the errors it raises."""
import sys

import pytest
import torch

import paper_2503_00540_amd as package
from paper_2503_00540_amd import rekv


@pytest.fixture
def fresh(monkeypatch):
    """The module as before its first use of the library."""
    rekv.lib()
    monkeypatch.setattr(rekv, "_lib", rekv._lib)
    monkeypatch.setattr(rekv, "_native", rekv._native)
    rekv._lib = rekv._native = None
    yield monkeypatch
    monkeypatch.undo()
    rekv._lib = None
    rekv.lib()


def test_a_refused_call_names_its_error_while_the_module_reloads_its_library(fresh):
    from paper_2503_00540_amd import _binding
    raising = []
    fresh.setattr(_binding, "set_raise", raising.append)
    rekv.lib()
    rekv._lib = None                                  # as __graft_entry__.build() leaves it before it loads the library again
    with pytest.raises(rekv.RekvError, match="REKV_ERR_INVALID_ARG"):
        raising[0](1, 0)


def test_the_library_loads_without_the_native_half(fresh):
    fresh.setitem(sys.modules, "paper_2503_00540_amd._binding", None)      # an import of it fails
    fresh.delattr(package, "_binding", raising=False)
    with pytest.warns(RuntimeWarning, match="does not load"):
        L = rekv.lib()

    def create(shape, handle):
        handle._obj.value = 1
        return 0

    fresh.setattr(L, "rekv_create", create)
    fresh.setattr(L, "rekv_destroy", lambda h: None)
    r = rekv.Rekv(4, 1, 64, 16, "f32")
    assert r._fast.encode_chunk(None, None, None, 0, 1, 1, 0, None) is None   # left to the Python method
    with pytest.raises(ValueError, match="k is shorter"):
        r.frame_keys(torch.zeros(3, 1, 64), 1)
    r.close()
