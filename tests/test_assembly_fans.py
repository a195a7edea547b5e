"""A dof that many elements share (a fan of prisms round one vertex): its row of the
global matrix is far longer than what LDS holds, and its pieces are taken side by
side.  The sums are those of the host in colour order, bit for bit, and the time
grows with the fan's size, not with its square: from 500 to 4000 elements 8 times the
work; one list per piece, one piece after the other, would be 64."""
import numpy as np
import pytest

from gpu_util import flush

pytestmark = pytest.mark.gpu


def _fan(ne, n):
    ids = 1 + np.arange(ne * (n - 1)).reshape(ne, n - 1)
    return np.concatenate([np.zeros((ne, 1)), ids], axis=1).astype(np.int32), 1 + ne * (n - 1)


@pytest.mark.parametrize("form", ["fp64", "fp32"])
@pytest.mark.parametrize("p,ne", [(1, 25), (1, 26), (1, 51), (1, 900), (2, 400), (3, 26), (3, 27), (4, 50)])
def test_values(p, ne, form):
    import torch
    import paper_1310_1194_amd as F
    n = F.nshp(p)
    flush(f"[fan] p={p} ne={ne} {form}")
    dofs, ndof = _fan(ne, n)
    plan = F.AsmPlan(dofs, ndof)
    T = np.float64 if form == "fp64" else np.float32
    rng = np.random.default_rng(ne)
    A, b = rng.normal(size=(ne, n, n)).astype(T), rng.normal(size=(ne, n)).astype(T)
    v0, r0 = rng.normal(size=plan.nnz).astype(T), rng.normal(size=ndof).astype(T)
    row_ptr, _ = (x.cpu().numpy() for x in plan.pattern())
    for start in (False, True):
        values, rhs = (v0.copy(), r0.copy()) if start else (np.zeros(plan.nnz, T), np.zeros(ndof, T))
        for e in np.argsort(plan.colors(), kind="stable"):
            # row 0 holds every dof; the others dof 0 and their own element's, ascending
            values[0] += A[e, 0, 0]
            values[dofs[e, 1:]] += A[e, 0, 1:]
            rhs[dofs[e]] += b[e]
            for a in range(1, n):
                values[row_ptr[dofs[e, a]]:row_ptr[dofs[e, a]] + n] += A[e, a]
        dv, dr = torch.from_numpy(v0).cuda(), torch.from_numpy(r0).cuda()
        plan.assemble(torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda(), form, values=dv, rhs=dr, accumulate=start)
        torch.cuda.synchronize()
        assert np.array_equal(dv.cpu().numpy(), values) and np.array_equal(dr.cpu().numpy(), rhs)


def test_time_grows_with_the_fan():
    import torch
    import paper_1310_1194_amd as F
    ms = []
    for ne in (500, 4000):
        dofs, ndof = _fan(ne, 6)
        plan = F.AsmPlan(dofs, ndof)
        A, b = torch.zeros((ne, 6, 6), dtype=torch.float64, device="cuda"), torch.zeros((ne, 6), dtype=torch.float64, device="cuda")
        v, r = torch.empty(plan.nnz, dtype=torch.float64, device="cuda"), torch.empty(ndof, dtype=torch.float64, device="cuda")
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        best = 1e30
        for _ in range(4):
            e[0].record()
            plan.assemble(A, b, "fp64", values=v, rhs=r)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]))
        ms.append(best)
        plan.close()
    flush(f"[fan] 500: {ms[0]:.3f} ms, 4000: {ms[1]:.3f} ms")
    assert ms[1] < 24 * ms[0]
