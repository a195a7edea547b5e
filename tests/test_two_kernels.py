"""The default kernels at p = 2, one for small batches and one for larger ones: on
both sides of the line, the bits of the kernel that the size calls for."""
import numpy as np
import pytest

from gpu_util import flush, to_dev
from paper_1310_1194_amd import meshgen

pytestmark = pytest.mark.gpu


# form, rule, elements up to which the first kernel runs, the kernels, whether
# coefficients at the vertices take the first at any size
@pytest.mark.parametrize("form,rule,line,name,few,many,fields_few", [
    ("fp32", "collapsed", 16384, "v18o4", "0x2fo4", "v18o2", True),
    ("bf16x3", "collapsed", 1024, "2x2so4", "2x2s", "0x2fo4", False),
    ("fp16x3", "collapsed", 1024, "2x2so4", "2x2s", "0x2fo4", False),
    ("bf16x3", "symmetric", 4096, "2x2so4", "2x2s", "0x2fo4", False),
    ("fp16x3", "symmetric", 2048, "2x2so4", "2x2s", "0x2fo4", False)])
def test_line(form, rule, line, name, few, many, fields_few):
    import torch
    import paper_1310_1194_amd as F
    names = [F.tile_describe(2, form, t, rule) for t in range(F.tile_count(2, form, rule))]
    assert names[0] == name and len(set(names)) == len(names)
    whole = meshgen.make_batch(32, 32, 9, amp=0.2, seed=5)
    for ne in (line, line + 1):
        X = to_dev(whole.subset(np.arange(ne)))
        fl = [torch.from_numpy(v).cuda() for v in meshgen.vertex_fields(ne, 6)]
        for fields in (False, True):
            def run(tile):
                flush(f"[two kernels] {form} {rule} ne={ne} fields={fields} {names[tile]}")
                F.tile_set(2, form, tile, rule)
                out = (F.integrate_fields_raw(X[0], *fl, 2, form, rule=rule) if fields else
                       F.integrate_raw(*X, 2, form, rule=rule))
                torch.cuda.synchronize()
                F.tile_set(2, form, 0, rule)
                return out
            want = few if ne <= line or (fields and fields_few) else many
            other = many if want == few else few
            A, b = run(0)
            Aw, bw = run(names.index(want))
            assert torch.equal(A, Aw) and torch.equal(b, bw)
            assert not torch.equal(A, run(names.index(other))[0])


@pytest.mark.parametrize("form", ["fp64", "fp32"])
def test_lanes_per_element_on_the_symmetric_rule(form):
    import paper_1310_1194_amd as F
    assert F.tile_describe(2, form, 0, "symmetric") == "v18o2"
