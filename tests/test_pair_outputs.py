"""The pair products' copies of A leave in 16-byte pieces from whatever address the
caller gives: outputs that start 1, 2 or 3 values into a buffer are the same, bit
for bit, as an aligned batch's, and nothing beside them is written.
"""
import numpy as np
import pytest

from gpu_util import flush, to_dev
from paper_1310_1194_amd import costmodel, meshgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,form", [(p, form) for form in ("fp64", "fp32", "bf16x3") for p in range(2 if form == "bf16x3" else 3, 8)])
def test_unaligned_outputs(p, form):
    import torch
    import paper_1310_1194_amd as F
    F.tile_set(p, form, next(t for t in range(F.tile_count(p, form)) if costmodel.is_pair_tile(F.tile_describe(p, form, t))))
    ne, n = 7, F.nshp(p)
    batch = meshgen.make_batch(4, 3, 1, amp=0.2, seed=p).subset(np.arange(ne))
    args = to_dev(batch)
    T = torch.float64 if form == "fp64" else torch.float32
    A0, b0 = torch.empty((ne, n, n), dtype=T, device="cuda"), torch.empty((ne, n), dtype=T, device="cuda")
    F.integrate_raw(*args, p, form, A=A0, b=b0)
    for off in (1, 2, 3):
        flush(f"[unaligned outputs] p={p} {form} off={off}")
        buf = torch.full((ne * n * n + 8,), 7.0, dtype=T, device="cuda")
        A = buf[off:off + ne * n * n].view(ne, n, n)
        F.integrate_raw(*args, p, form, A=A, b=b0)
        torch.cuda.synchronize()
        assert torch.equal(A, A0)
        assert (buf[:off] == 7.0).all() and (buf[off + ne * n * n:] == 7.0).all()
    F.tile_set(p, form, 0)
