"""A dof listed twice in one element is refused wherever it stands: neighbouring or
distant places of the element, the first or the last element, a dof that many
elements share, maps of one and of several host threads."""
import ctypes

import numpy as np
import pytest

from paper_1310_1194_amd import native


@pytest.mark.parametrize("ne,n", [(1, 6), (40, 18), (2000, 6)])
@pytest.mark.parametrize("places", [(0, 1), (0, -1), (2, 4)])
def test_repeated_dof(ne, n, places):
    ids = np.arange(ne * n, dtype=np.int32).reshape(ne, n)
    ids[1:, 3] = ids[0, 3]                                    # shared by all
    for e in {0, ne // 2, ne - 1}:
        for src in {places[0], 3}:
            d = ids.copy()
            dst = places[1] if places[1] % n != src else 5
            d[e, dst] = d[e, src]
            h = ctypes.c_void_p()
            assert native.lib().feint_asm_plan_create(d.ctypes.data_as(ctypes.c_void_p), ne, n, ne * n, ctypes.byref(h)) == -1
            assert not h.value
