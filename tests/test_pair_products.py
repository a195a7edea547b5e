"""The prisms' products of pairs of triangle functions ("0xWf" tiles).

CPU: the class sizes against a count of orbits and reflected points, the issued
matrix work against the algorithm's, the tile names.
GPU: element counts at the edges of a workgroup's share of elements, and one
that sends every workgroup of a full device on to a second and third group
(the inputs fetched ahead), on both rules and with vertex fields, against the
oracle; the det J flag and every mapped point in the same runs.

Tolerances: those of the forward parity tests, which are derived from the
forms' rounding and not from a kernel (fp64 1e-12, fp32 and fp16x3 2e-6, bf16x3
1e-5, relative Frobenius norm over the batch; per element 1e-12, 2e-5, 2e-5,
5e-5).
"""
import numpy as np
import pytest

import oracle
from paper_1310_1194_amd import costmodel, meshgen

TOL = {"fp64": (1e-12, 1e-12), "fp32": (2e-6, 2e-5), "bf16x3": (1e-5, 5e-5), "fp16x3": (2e-6, 2e-5)}


def _reflection(p):
    lattice = [(i, j) for j in range(p + 1) for i in range(p + 1 - j)]
    return [lattice.index((p - i - j, j)) for i, j in lattice]


@pytest.mark.parametrize("rule", ["collapsed", "symmetric"])
@pytest.mark.parametrize("p", range(1, 8))
def test_class_sizes(p, rule):
    st = _reflection(p)
    n = len(st)
    orbits = {frozenset({(a, b), (b, a), (st[a], st[b]), (st[b], st[a])}) for a in range(n) for b in range(n)}
    pts, _ = oracle.prism_rule(p, rule)
    tri = pts[: len(pts) // (p + 1), :2]
    mirror = np.stack([1 - tri.sum(1), tri[:, 1]], 1)
    image = [int(np.argmin(np.abs(tri - m).sum(1))) for m in mirror]
    assert np.abs(tri[image] - mirror).max() < 1e-12          # the rule is symmetric
    fixed = sum(i == q for q, i in enumerate(image))
    pairs = (len(tri) - fixed) // 2
    # an orbit has an entry in a class unless the class's combination of its four pairs vanishes
    rows = [0, 0, 0, 0]
    for o in orbits:
        a, b = min(o)
        for c in range(4):
            par, sym = (1 if c < 2 else -1), (1 if c % 2 == 0 else -1)
            total = {}
            for pair, w in (((a, b), 1), ((b, a), sym), ((st[a], st[b]), par), ((st[b], st[a]), par * sym)):
                total[pair] = total.get(pair, 0) + w
            rows[c] += any(total.values())
    sizes = costmodel.pair_sizes(p, rule)
    assert sizes[0] == (len(orbits), 6 * pairs + 4 * fixed)
    assert [k for _, k in sizes[1:]] == [3 * pairs + fixed, 6 * pairs + 2 * fixed, 3 * pairs + 2 * fixed]
    assert sum(rows) == n * n                                  # one result per pair (t, t')
    assert all(r <= s for r, (s, _) in zip(rows, sizes))       # rows past a class's own are table zeros
    assert sum(k for _, k in sizes) == 9 * len(tri)
    assert costmodel.pair_mfma_flops(p, rule) >= sum(2 * r * k for r, k in sizes) * (p + 1) ** 2
    assert costmodel.f_pair(p, rule) < costmodel.f_dom(p, rule)


def test_pair_tile_names():
    for d in ("0x4f", "0x4fo2", "0x8fo2"):
        assert costmodel.is_pair_tile(d) and not costmodel.is_kf_tile(d)
        assert costmodel.f_kernel(4, "collapsed", d) == costmodel.f_pair(4)
    assert not costmodel.is_pair_tile("4x4f") and not costmodel.is_pair_tile("5x3fo2")


# elements per workgroup and a count past two full devices' worth of workgroups (256 CUs, at most 8 each)
COUNTS = {2: (1, 4, 6, 21001), 3: (1, 3, 5, 16501), 4: (1, 2, 4201), 5: (1, 2103), 6: (1, 1031), 7: (1, 523)}


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["fp64", "fp32", "bf16x3", "fp16x3"])
@pytest.mark.parametrize("p", range(2, 8))
def test_pair_products_parity(p, form):
    import torch
    import paper_1310_1194_amd as F
    from gpu_util import flush, rel_errors, to_dev
    top = max(COUNTS[p])
    nz = max(2, round((top / 32) ** (1 / 3)))
    nx = int(np.ceil(np.sqrt(top / (2 * nz))))
    whole = meshgen.make_batch(nx, nx, nz, amp=0.2, seed=40 + p)
    for rule in ("collapsed", "symmetric"):
        tiles = [t for t in range(F.tile_count(p, form, rule)) if costmodel.is_pair_tile(F.tile_describe(p, form, t, rule))]
        if not tiles:                                          # p = 2 in FP64 and FP32
            continue
        F.tile_set(p, form, tiles[0], rule)
        for fields in (False, True):
            for ne in COUNTS[p] if rule == "collapsed" else COUNTS[p][-2:-1]:
                flush(f"[pair] p={p} {form} {rule} fields={fields} ne={ne}")
                batch = whole.subset(np.arange(ne) * (whole.ne // ne) if ne < 100 else np.arange(ne))
                check = np.arange(ne) if ne < 100 else np.r_[0:8, ne // 2:ne // 2 + 8, ne - 8:ne]
                sub = batch.subset(check)
                X = to_dev(batch)
                xq = torch.full((ne, F.nq(p, rule), 3), float("nan"), dtype=torch.float64, device="cuda")
                status = torch.zeros(1, dtype=torch.int32, device="cuda")
                rl = None if rule == "collapsed" else rule
                if fields:
                    fl = meshgen.vertex_fields(ne, 50 + p)
                    A, b = F.integrate_fields_raw(X[0], *[torch.from_numpy(v).cuda() for v in fl], p, form, xq=xq,
                                                  status=status, rule=rule)
                    Ar, br, _, xr = oracle.integrate_fields(p, sub.coords, *[np.ascontiguousarray(v[check]) for v in fl],
                                                         want_xq=True, rule=rl)
                else:
                    A, b = F.integrate_raw(*X, p, form, xq=xq, status=status, rule=rule)
                    Ar, br, _, xr = oracle.integrate(p, sub.coords, sub.D, sub.beta, sub.c, sub.f, want_xq=True, rule=rl)
                torch.cuda.synchronize()
                ids = torch.from_numpy(check).cuda()
                gA, mA = rel_errors(A[ids].cpu().numpy(), Ar)
                gb, mb = rel_errors(b[ids].cpu().numpy(), br)
                assert gA < TOL[form][0] and mA < TOL[form][1], (gA, mA)
                assert gb < TOL[form][0] and mb < TOL[form][1], (gb, mb)
                assert np.abs(xq[ids].cpu().numpy().reshape(len(check), -1, 3) - xr.reshape(len(check), -1, 3)).max() < 1e-14
                assert torch.isfinite(A).all() and torch.isfinite(b).all() and torch.isfinite(xq).all()
                assert int(status.item()) == 0
        F.tile_set(p, form, 0, rule)
