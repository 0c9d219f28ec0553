"""float32 kernels at the edges of their tiles against the CPU oracle: k ranges that end inside a step of sixteen, columns
that end inside a tile, one to four row tiles per workgroup, both head sizes, contexts shorter than the four waves'
shares."""
import numpy as np
import pytest

import workloads as wl
import paper_2504_04104_amd as sp
from gpu_harness import Pair, rel_err

pytestmark = pytest.mark.gpu

SHAPES = {"d264_h64": wl.ModelShape(n_layers=2, d_model=264, n_q_heads=3, n_kv_heads=1, d_head=64, d_ff=104, rms_eps=1e-6, dtype="f32"),
          "d72_h128": wl.ModelShape(n_layers=2, d_model=72, n_q_heads=4, n_kv_heads=2, d_head=128, d_ff=40, rms_eps=1e-6, dtype="f32")}


@pytest.mark.parametrize("page_slots", [0, 32], ids=["contiguous", "pages32"])
@pytest.mark.parametrize("n,prefix", [(1, 1), (3, 2), (17, 200), (40, 63), (70, 300)])
@pytest.mark.parametrize("shape", SHAPES.values(), ids=SHAPES.keys())
def test_f32_tiles(shape, n, prefix, page_slots):
    """The increment within 2e-5 of its largest value: sums of up to 264 products and 370 slots in float32 (unit roundoff
    6e-8, errors grow with the root of the count to some 1e-6) and exponentials good to about 2e-7 per unit of their
    argument, on trees whose last levels have ancestors all over the range.  Three calls: the later ones replay."""
    pair = Pair(shape, 29, {0: prefix}, max_batch_nodes=80, page_slots=page_slots)
    pair.insert(0, wl.tree_deep(29, n, 20))
    for k in range(3):
        x = wl.hidden_rows(shape, 29, ("f32", n, k), n)
        y, ref = pair.forward([0], [0], [n], x)
        e = rel_err(y - x, ref - x)
        print(n, prefix, e, flush=True)
        assert e <= 2e-5
    pair.check_kv(0, 2e-5)
    pair.close()
