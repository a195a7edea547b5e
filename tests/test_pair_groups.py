"""Pair-product kernels whose workgroups go on to second and third groups of elements
(the inputs fetched ahead, the zeta sums, E and A overlapping in LDS, the turn of
the waves): the symmetric rule, whose LDS extents are its own, with
coefficients per element and per vertex, and the Laplace term.  Every element
against another kernel, some against the oracle; and which (p, form, rule) have
such a kernel.

Tolerances: those of the forward parity tests (fp64 1e-12, fp32 and fp16x3 2e-6,
bf16x3 1e-5 over the batch; per element 1e-12, 2e-5, 2e-5, 5e-5), twice that
between two kernels.
"""
import numpy as np
import pytest

import oracle
from gpu_util import flush, rel_errors, to_dev
from paper_1310_1194_amd import costmodel, meshgen

pytestmark = pytest.mark.gpu

TOL = {"fp64": (1e-12, 1e-12), "fp32": (2e-6, 2e-5), "bf16x3": (1e-5, 5e-5), "fp16x3": (2e-6, 2e-5)}
# elements past two full devices' worth of workgroups (256 CUs, at most 8 each)
COUNT = {2: 21001, 3: 16501, 4: 4201, 5: 2103, 6: 1031, 7: 523}


def _batch(p, seed):
    ne = COUNT[p]
    nz = max(2, round((ne / 32) ** (1 / 3)))
    nx = int(np.ceil(np.sqrt(ne / (2 * nz))))
    return meshgen.make_batch(nx, nx, nz, amp=0.2, seed=seed).subset(np.arange(ne))


def _close(got, want, tol):
    """Over the batch, and element by element, in the norm of the second."""
    got, want = got.double().flatten(1), want.double().flatten(1)
    d, n = (got - want).norm(dim=1), want.norm(dim=1)
    assert float(d.norm() / n.norm()) < 2 * tol[0] and float((d / n).max()) < 2 * tol[1]


@pytest.mark.parametrize("form", ["fp64", "fp32", "bf16x3", "fp16x3"])
@pytest.mark.parametrize("p", range(2, 8))
def test_symmetric_rule(p, form):
    import torch
    import paper_1310_1194_amd as F
    names = [F.tile_describe(p, form, t, "symmetric") for t in range(F.tile_count(p, form, "symmetric"))]
    pair = [t for t, d in enumerate(names) if costmodel.is_pair_tile(d)]
    assert len(pair) == (0 if p == 2 and form in ("fp64", "fp32") else 1)
    assert len([t for t in range(F.tile_count(p, form)) if costmodel.is_pair_tile(F.tile_describe(p, form, t))]) == (
        0 if p == 2 and form == "fp64" else 1)
    if not pair:
        return
    batch = _batch(p, 80 + p)
    ne = batch.ne
    check = np.r_[0:6, ne // 2:ne // 2 + 6, ne - 6:ne]
    sub, ids = batch.subset(check), torch.from_numpy(check).cuda()
    X, fl = to_dev(batch), meshgen.vertex_fields(ne, 90 + p)
    dfl = [torch.from_numpy(v).cuda() for v in fl]
    for fields in (False, True):
        flush(f"[groups] p={p} {form} {names[pair[0]]} ne={ne} fields={fields}")
        out = []
        for tile in (pair[0], pair[0] + 1):
            F.tile_set(p, form, tile, "symmetric")
            out.append(F.integrate_fields_raw(X[0], *dfl, p, form, rule="symmetric") if fields else
                       F.integrate_raw(*X, p, form, rule="symmetric"))
        F.tile_set(p, form, 0, "symmetric")
        torch.cuda.synchronize()
        (A, b), (A2, b2) = out
        if fields:
            Ar, br, _ = oracle.integrate_fields(p, sub.coords, *[np.ascontiguousarray(v[check]) for v in fl], rule="symmetric")
        else:
            Ar, br, _ = oracle.integrate(p, sub.coords, sub.D, sub.beta, sub.c, sub.f, rule="symmetric")
        for got, other, ref in ((A, A2, Ar), (b, b2, br)):
            g, m = rel_errors(got[ids].cpu().numpy(), ref)
            assert g < TOL[form][0] and m < TOL[form][1], (g, m)
            _close(got, other, TOL[form])


@pytest.mark.parametrize("form", ["fp64", "fp32"])
@pytest.mark.parametrize("p", range(3, 8))
def test_laplace(p, form):
    import torch
    import paper_1310_1194_amd as F
    names = [F.laplace_tile_describe(p, form, t) for t in range(F.laplace_tile_count(p, form))]
    pair = [t for t, d in enumerate(names) if costmodel.is_pair_tile(d)]
    assert len(pair) == 1
    batch = _batch(p, 60 + p)
    ne = batch.ne
    check = np.r_[0:6, ne // 2:ne // 2 + 6, ne - 6:ne]
    X = torch.from_numpy(batch.coords).cuda()
    flush(f"[groups] laplace p={p} {form} {names[pair[0]]} ne={ne}")
    out = []
    for tile in (pair[0], pair[0] + 1):
        F.laplace_tile_set(p, form, tile)
        out.append(F.integrate_laplace_raw(X, p, form))
    F.laplace_tile_set(p, form, 0)
    torch.cuda.synchronize()
    Ar, _ = oracle.integrate_laplace(p, batch.coords[check])
    g, m = rel_errors(out[0][torch.from_numpy(check).cuda()].cpu().numpy(), Ar)
    assert g < TOL[form][0] and m < TOL[form][1], (g, m)
    _close(out[0], out[1], TOL[form])
