"""What the binding does with the library's answers (no GPU: a stand-in for the
library)."""
import ctypes
import types

import numpy as np
import pytest

from paper_2507_14813_amd import api


class EnumerateTwice:
    """mg_enumerate and mg_enumerate_arrays whose two searches find `first` and
    `second` matches."""

    def __init__(self, first, second):
        self.first, self.second = first, second

    def mg_enumerate(self, g, t, st, out, capacity, n):
        n._obj.value = self.first
        return 0

    def mg_enumerate_arrays(self, g, t, st, motif, edges, capacity, n):
        n._obj.value = self.second
        if self.second <= capacity:
            ctypes.memset(motif, 0, 4 * self.second)
            ctypes.memset(edges, 255, 20 * self.second)
        return 0


@pytest.mark.parametrize("first,second", [(0, 0), (3, 3), (3, 2), (3, 4), (3, 0)])
def test_enumerated_matches_are_all_or_an_error(monkeypatch, first, second):
    monkeypatch.setattr(api, "lib", lambda: EnumerateTwice(first, second))
    handle = types.SimpleNamespace(handle=ctypes.c_void_p(1))
    if first != second:
        with pytest.raises(api.MayuraError, match="MG_EINTERNAL"):
            api.enumerate_matches(handle, handle, stream=0)
        return
    motif, edges = api.enumerate_matches(handle, handle, stream=0)
    assert motif.shape == (first,) and edges.shape == (first, 5)
    assert np.all(motif == 0) and np.all(edges == -1)
