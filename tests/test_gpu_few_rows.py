"""The kernels for one row tile (1-16 rows: complete projections with RoPE, cache append, residual, norm and
write-out as their epilogues) against the CPU oracle, at the k lengths that select each number of fragments in flight."""
import numpy as np
import pytest
import torch

import workloads as wl
import paper_2504_04104_amd as sp
from gpu_harness import Pair, rel_err, to_dev, to_np

pytestmark = pytest.mark.gpu

# k steps per wave: 8 / 8 / 16 (eight fragments in flight), 2 / 4 / 6 (two), 3 / 4 / 5 (one and two)
SHAPES = {"k2048": wl.ModelShape(n_layers=2, d_model=2048, n_q_heads=16, n_kv_heads=4, d_head=128, d_ff=4096),
          "k512": wl.ModelShape(n_layers=2, d_model=512, n_q_heads=8, n_kv_heads=8, d_head=128, d_ff=1536),
          # 8192 columns in O and down: two strips per workgroup; 16 rows, and 6 row-major: split products
          "n8192": wl.ModelShape(n_layers=2, d_model=8192, n_q_heads=16, n_kv_heads=2, d_head=128, d_ff=2048),
          "k768": wl.ModelShape(n_layers=2, d_model=768, n_q_heads=8, n_kv_heads=1, d_head=128, d_ff=1280)}


@pytest.mark.parametrize("page_slots", [0, 32], ids=["contiguous", "pages32"])
@pytest.mark.parametrize("packed", [True, False], ids=["packed", "rowmajor"])
@pytest.mark.parametrize("n", [1, 6, 16])
@pytest.mark.parametrize("shape", SHAPES.values(), ids=SHAPES.keys())
def test_one_row_tile(shape, n, packed, page_slots):
    """Increment and cache rows against the oracle (bf16 bar: 2e-2 of the largest value), then the same call again with
    other inputs into other tensors, in place at last: a replayed call has to write where that call says and nowhere
    else."""
    pair = Pair(shape, 71, {0: 45}, flags=sp.SP_FLAG_PACKED_WEIGHTS if packed else 0, page_slots=page_slots)
    pair.insert(0, wl.tree_deep(71, n, 9))
    outs = []
    for k in range(4):
        x = wl.hidden_rows(shape, 71, ("few", n, k), n)
        xd = to_dev(x, pair.gpu)
        y = xd if k == 3 else torch.full_like(xd, float("nan"))
        pair.gpu.stage_forward([0], [0], [n], xd, y)
        ref = pair.ora.stage_forward(0, 0, x)
        outs.append((y, to_np(y)))
        assert rel_err(outs[-1][1] - x, ref - x) <= 2e-2, k
        pair.check_kv(0, 2e-2)
    for y, seen in outs:
        assert np.array_equal(to_np(y), seen)
    pair.close()
