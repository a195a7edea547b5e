"""The launches per degree of a mixed batch: batches on both sides of the count
at which FP64 takes the single persistent launch, degrees missing from the
batch, and one past a device's worth of workgroups, against the oracle.

Tolerances: those of the mixed parity tests (fp64 1e-12, fp32 2e-6, relative
Frobenius norm per degree).
"""
import numpy as np
import pytest

import oracle
from gpu_util import flush, rel_errors, to_dev
from paper_1310_1194_amd import meshgen

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 2e-6}


@pytest.mark.parametrize("form", ["fp64", "fp32"])
@pytest.mark.parametrize("ne,degrees", [(1, (3,)), (512, (1, 2, 3, 4, 5, 6)), (513, (1, 2, 3, 4, 5, 6)), (700, (2, 5)),
                                        (9001, (1, 3, 3, 3, 4))])
def test_bucket_launches(ne, degrees, form):
    import torch
    import paper_1310_1194_amd as F
    rng = np.random.default_rng(ne)
    batch = meshgen.make_batch(32, 32, 8, amp=0.2, seed=ne).subset(np.arange(ne))
    deg = rng.choice(np.array(degrees), ne).astype(np.int8)
    X = to_dev(batch)
    plan = F.MixedPlan(ne, form)
    offA, offb = plan.bucket(torch.from_numpy(deg).cuda())
    A, b = plan.alloc_outputs(offA, offb)
    A.fill_(float("nan"))
    b.fill_(float("nan"))
    flush(f"[buckets] {form} ne={ne} degrees={degrees}")
    plan.integrate(*X, A, b, offA, offb)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(A).all()) and bool(torch.isfinite(b).all())
    oA, ob, A, b = offA.cpu().numpy(), offb.cpu().numpy(), A.cpu().numpy(), b.cpu().numpy()
    for d in sorted(set(degrees)):
        ids = np.nonzero(deg == d)[0]
        ids = np.unique(np.r_[ids[:6], ids[-6:]])
        sub = batch.subset(ids)
        Ar, br, _ = oracle.integrate(d, sub.coords, sub.D, sub.beta, sub.c, sub.f)
        n = Ar.shape[1]
        gA, _ = rel_errors(np.stack([A[oA[e]:oA[e] + n * n] for e in ids]), Ar)
        gb, _ = rel_errors(np.stack([b[ob[e]:ob[e] + n] for e in ids]), br)
        assert gA < TOL[form] and gb < TOL[form], (d, gA, gb)
    plan.close()
