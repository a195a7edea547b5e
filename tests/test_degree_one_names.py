"""The kernels of prisms of degree 1: a description each, and the work of the one from
moments against a count of the loops that it runs."""
import pytest

from paper_1310_1194_amd import costmodel, native

import ctypes


@pytest.mark.parametrize("rule", [0, 1])
@pytest.mark.parametrize("form", [0, 1])
def test_names_differ(form, rule):
    L, buf = native.lib(), ctypes.create_string_buffer(32)
    names = []
    for t in range(L.feint_rule_tile_count(1, form, rule)):
        assert L.feint_rule_tile_describe(1, form, rule, t, buf, 32) == 0
        names.append(buf.value.decode())
    assert names[0] == "v1o2" and len(set(names)) == len(names)


@pytest.mark.parametrize("rule", ["collapsed", "symmetric"])
def test_work_from_moments(rule):
    flops = 0
    for _ in range(2):                                        # zeta points
        for _ in range(costmodel.nq(1, rule) // 2):           # triangle points
            flops += 4                                        # oo, ee, oe + eo, oe - eo
            for i in range(3):
                flops += 2 * (6 + 1)                          # l_i times 0o 0e o3 e3 3o 3e, w det J f
                for j in range(i, 3):
                    flops += 1 + 2 * 3                        # l_i l_j times 00, 03, 33
        flops += 4 * 4                                        # products of line factors of (k, k')
        oe = (2, 2, 0)                                        # T_o(t) o + T_e(t) e
        for i in range(3):
            for j in range(3):
                flops += 2 + oe[j] + oe[i] + 2 * oe[j]        # P
                flops += 1 + oe[i]                            # Q
                flops += oe[j]                                # R
                flops += 4 * (1 + 3 * 2 + 1)                  # (k, k'), the sum over zeta points
        flops += 6 * 2                                        # load vector
    assert costmodel.f_moments(rule) == flops == costmodel.f_kernel(1, rule, "v1o2")
    assert costmodel.f_kernel(1, rule, "v1") == costmodel.f_dom(1, rule) > flops
