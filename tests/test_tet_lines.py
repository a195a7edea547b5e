"""Tetrahedra whose element matrices leave in whole lines ("ref2s"): the products are
those of the other reference-matrix kernels, so every entry is the same bit for bit
wherever the output starts in a line, at full waves, ragged tails and single elements,
and nothing beside the output is written.
"""
import numpy as np
import pytest

from gpu_util import flush
from paper_1310_1194_amd import meshgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,form", [(3, "fp32"), (4, "fp32"), (6, "fp32"), (3, "fp64"), (4, "fp64")])
def test_whole_lines(p, form):
    import torch
    import paper_1310_1194_amd as F
    T = torch.float64 if form == "fp64" else torch.float32
    names = [F.elem_tile_describe("tet", p, form, t) for t in range(F.elem_tile_count("tet", p, form))]
    lines = [t for t, s in enumerate(names) if s.startswith("ref2s") and s.endswith("o4")]
    assert lines and names.index("ref1o2") >= 0
    n = F.tet_nshp(p)
    whole = meshgen.make_tet_batch(4, 4, 3, amp=0.2, seed=p)
    for ne in (1, 16, 64, 81, 200):
        b = whole.subset(np.arange(ne))
        X = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (b.coords, b.D, b.beta, b.c, b.f)]
        F.elem_tile_set("tet", p, form, names.index("ref1o2"))
        A0, b0 = F.integrate_elem_raw("tet", *X, p, form)
        for t in lines + [0]:
            F.elem_tile_set("tet", p, form, t)
            for off in (0, 1, 3, 31):
                flush(f"[tet lines] p={p} {form} {names[t]} ne={ne} off={off}")
                buf = torch.full((ne * n * n + 64,), 7.0, dtype=T, device="cuda")
                A = buf[off:off + ne * n * n].view(ne, n, n)
                b1 = torch.empty_like(b0)
                F.integrate_elem_raw("tet", *X, p, form, A=A, b=b1)
                torch.cuda.synchronize()
                assert torch.equal(A, A0) and torch.equal(b1, b0)
                assert (buf[:off] == 7.0).all() and (buf[off + ne * n * n:] == 7.0).all()
    F.elem_tile_set("tet", p, form, 0)
