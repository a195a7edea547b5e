"""Assembly row by row at the sizes where its loops end: fans of elements that all
share one dof (a row longer than what LDS holds at once, more element rows than
lanes), every split of an element row over the lanes, single elements, and dofs
that no element has.  The sums are made in colour order, so the values are those
of the same additions on the host, bit for bit.
"""
import numpy as np
import pytest

from gpu_util import flush

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["fp64", "fp32"])
@pytest.mark.parametrize("more", [0, 66000])     # rows without elements; several rows per wave from 65536 on
@pytest.mark.parametrize("p,ne", [(1, 1), (1, 47), (2, 45), (3, 70), (4, 33), (5, 3), (6, 9), (7, 5)])
def test_fan(p, ne, more, form):
    import torch
    import paper_1310_1194_amd as F
    n = F.nshp(p)
    flush(f"[assembly rows] p={p} ne={ne} more={more} {form}")
    rng = np.random.default_rng(p * 100 + ne)
    # dof 5 is shared by all, dof 3 by none, two more by neighbours
    ids = 6 + rng.permutation(ne * (n - 1)).reshape(ne, n - 1)
    ids[1:, 0] = ids[:-1, 1]
    dofs = np.concatenate([ids, np.full((ne, 1), 5)], axis=1).astype(np.int32)
    dofs = np.stack([rng.permutation(r) for r in dofs])
    ndof = 6 + ne * (n - 1) + more
    plan = F.AsmPlan(dofs, ndof)
    T = np.float64 if form == "fp64" else np.float32
    A, b = rng.normal(size=(ne, n, n)).astype(T), rng.normal(size=(ne, n)).astype(T)
    dA, db = torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda()
    row_ptr, col = (x.cpu().numpy() for x in plan.pattern())
    order = np.argsort(plan.colors(), kind="stable")
    place = {}
    for i in np.unique(dofs):
        place[i] = {c: k for k, c in zip(range(row_ptr[i], row_ptr[i + 1]), col[row_ptr[i]:row_ptr[i + 1]])}
    for start in (False, True):
        v0, r0 = rng.normal(size=plan.nnz).astype(T), rng.normal(size=ndof).astype(T)
        values, rhs = (v0.copy(), r0.copy()) if start else (np.zeros(plan.nnz, T), np.zeros(ndof, T))
        for e in order:
            for a in range(n):
                at = place[dofs[e, a]]
                values[[at[c] for c in dofs[e]]] += A[e, a]
            rhs[dofs[e]] += b[e]
        dv, dr = torch.from_numpy(v0).cuda(), torch.from_numpy(r0).cuda()
        plan.assemble(dA, db, form, values=dv, rhs=dr, accumulate=start)
        torch.cuda.synchronize()
        assert np.array_equal(dv.cpu().numpy(), values)
        assert np.array_equal(dr.cpu().numpy(), rhs)
