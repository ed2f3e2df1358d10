"""Without the extension module (not built, or built against another torch)
the Python functions make every call themselves, after a warning."""
import sys

import pytest
import torch

import paper_1809_09851_amd
from paper_1809_09851_amd import fdbb as F


@pytest.fixture
def no_module(monkeypatch):
    lib = F.library()
    monkeypatch.setitem(sys.modules, "paper_1809_09851_amd._binding", None)
    monkeypatch.delattr(paper_1809_09851_amd, "_binding", raising=False)
    with pytest.warns(RuntimeWarning, match="native binding"):
        F._bind(lib)
    yield
    monkeypatch.undo()
    F._bind(lib)


def test_calls_go_through_the_library(no_module):
    U, V = torch.ones(3, 8, dtype=torch.float64), torch.empty(3, 8, dtype=torch.float64)
    with pytest.raises(ValueError, match="device memory"):
        F.fdbb_cons2prim(1, 1.4, U, V)
    assert F._run(0) is None and F._char_apply(0) is None and F._viscous_flux(0) is None
    assert F._fields_like(4, U).shape == (4, 8) and F._blocks_like(1, U).shape == (1, 8, 3, 3)


def test_module_is_used_where_it_is_there():
    F.library()
    from paper_1809_09851_amd import _binding
    assert F._run is _binding.run and F._empty_fields is _binding.empty_fields
