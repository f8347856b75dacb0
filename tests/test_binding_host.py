"""The native half of the binding as far as it goes without a GPU: loading it, and the errors it raises."""
import pytest

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
