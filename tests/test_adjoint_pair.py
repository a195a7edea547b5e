"""The FP64 adjoint through the products of pairs of triangle functions (block
"0xWf"): element counts below, at and above a workgroup's share, both rules,
against the oracle's reverse-mode gradient.

Tolerances: those of the adjoint parity tests (1e-11 global, 1e-10 per element
relative to its own norm, floored at 1e-2 of the batch's).  No global atomics
take part, so two runs agree bit for bit.
"""
import numpy as np
import pytest

import oracle
from gpu_util import flush, grad_errors, to_dev
from paper_1310_1194_amd import costmodel, meshgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rule", ["collapsed", "symmetric"])
@pytest.mark.parametrize("p", range(3, 8))
def test_adjoint_pair(p, rule):
    import torch
    import paper_1310_1194_amd as F
    tile = [t for t in range(F.adjoint_tile_count(p, "fp64"))
            if costmodel.is_pair_tile(F.adjoint_tile_describe(p, "fp64", t))][0]
    F.adjoint_tile_set(p, "fp64", tile)
    n = F.nshp(p)
    rng = np.random.default_rng(60 + p)
    for ne in (1, 2, 5, 300):
        batch = meshgen.make_batch(13, 12, 1, amp=0.2, seed=p).subset(np.arange(ne))
        G, g = rng.normal(size=(ne, n, n)), rng.normal(size=(ne, n))
        flush(f"[adjoint pair] p={p} {rule} ne={ne}")
        args = [*to_dev(batch), torch.from_numpy(G).cuda(), torch.from_numpy(g).cuda()]
        got = F.adjoint_raw(*args, p, "fp64", rule=rule)
        again = F.adjoint_raw(*args, p, "fp64", rule=rule)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, again))
        ids = np.unique(np.r_[0:min(ne, 4), max(0, ne - 4):ne])
        sub = batch.subset(ids)
        ref = oracle.adjoint(p, sub.coords, sub.D, sub.beta, sub.c, sub.f, np.ascontiguousarray(G[ids]),
                             np.ascontiguousarray(g[ids]), rule=None if rule == "collapsed" else rule)
        for name, a, r in zip(("dcoords", "dD", "dbeta", "dc", "df"), got, ref):
            gl, el = grad_errors(a.cpu().numpy()[ids], r, floor=1e-2)
            assert gl <= 1e-11 and el <= 1e-10, (name, gl, el)
    F.adjoint_tile_set(p, "fp64", 0)
