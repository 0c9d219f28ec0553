"""The kernels for one row tile (1-16 rows: complete projections with RoPE, cache append, residual, norm and
write-out as their epilogues) against the CPU oracle, at the k lengths that select each number of fragments in flight."""
import numpy as np
import pytest
import torch

import workloads as wl
import paper_2504_04104_amd as sp
from gpu_harness import Pair, rel_err, to_dev, to_np

pytestmark = pytest.mark.gpu

SP_K_ROPE_KV = 11          # sp_kernel_kind

# k steps per wave: 8 / 8 / 16 (eight fragments in flight), 2 / 4 / 6 (two), 3 / 4 / 5 (one and two)
SHAPES = {"k2048": wl.ModelShape(n_layers=2, d_model=2048, n_q_heads=16, n_kv_heads=4, d_head=128, d_ff=4096),
          "k512": wl.ModelShape(n_layers=5, d_model=512, n_q_heads=8, n_kv_heads=8, d_head=128, d_ff=1536),
          # 8192 columns in O and down: two strips per workgroup; 16 rows, and all of row-major: split products
          "n8192": wl.ModelShape(n_layers=2, d_model=8192, n_q_heads=16, n_kv_heads=2, d_head=128, d_ff=2048),
          "k768": wl.ModelShape(n_layers=5, d_model=768, n_q_heads=8, n_kv_heads=1, d_head=128, d_ff=1280)}


@pytest.mark.parametrize("page_slots", [0, 32], ids=["contiguous", "pages32"])
@pytest.mark.parametrize("packed", [True, False], ids=["packed", "rowmajor"])
@pytest.mark.parametrize("n", [1, 6, 16])
@pytest.mark.parametrize("shape", SHAPES.values(), ids=SHAPES.keys())
def test_one_row_tile(shape, n, packed, page_slots):
    """Increment and cache rows against the oracle (bf16 bar: 2e-2 of the largest value), then the same call again with
    other inputs into other tensors, in place at last: every call has to write where it says and nowhere else, also where it
    replays a graph (five layers: at least 25 launches; two are made one by one)."""
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


# shape, weights, [(rows, complete projections?)]
ROUTES = [
    # up to one workgroup per CU in O and down, whole rounds (8192: two strips each), else up to four rows
    ("d4096", (4096, 32, 8, 512), True, [(16, True)]),
    ("d8192", (8192, 16, 2, 512), True, [(12, True), (13, False)]),
    ("d4608", (4608, 36, 4, 512), True, [(4, True), (5, False), (16, False)]),
    # row-major weights: up to 4096 columns, and rows by their length
    ("d4096", (4096, 32, 8, 512), False, [(8, True), (9, False)]),
    ("d4608", (4608, 36, 4, 512), False, [(1, False)]),
    # an odd number of k steps per wave leaves one load in flight: only short k ranges
    ("ff8960", (512, 4, 2, 8960), True, [(1, False)]),
    # ... with QKV's 192 tiles in four slices (three workgroups per CU), O and down in sixteen
    ("mha", (1024, 32, 32, 8960), True, [(1, False), (16, False)]),
    ("mha", (1024, 32, 32, 8960), False, [(9, False)]),
    ("ff1792", (512, 4, 2, 1792), True, [(16, True)]),
]


@pytest.mark.parametrize("name,dims,packed,calls", ROUTES, ids=[f"{r[0]}_{'packed' if r[2] else 'rowmajor'}" for r in ROUTES])
def test_which_rows_take_complete_projections(name, dims, packed, calls):
    """Where the line between complete and split projections lies (a call with complete ones has no RoPE launch of its
    own), and results on both of its sides against the oracle."""
    d, nq, nkv, ff = dims
    shape = wl.ModelShape(n_layers=1, d_model=d, n_q_heads=nq, n_kv_heads=nkv, d_head=128, d_ff=ff)
    pair = Pair(shape, 37, {r: 30 for r in range(len(calls))}, flags=sp.SP_FLAG_PACKED_WEIGHTS if packed else 0)
    for r, (n, complete) in enumerate(calls):
        pair.insert(r, wl.tree_deep(37 + n, n, 7))
        x = wl.hidden_rows(shape, 37, ("route", n), n)
        pair.gpu.profile_begin(SP_K_ROPE_KV, 4)
        y, ref = pair.forward([r], [0], [n], x)
        launches, _ = pair.gpu.profile_end()
        assert (launches == 0) == complete, (n, launches)
        assert rel_err(y - x, ref - x) <= 2e-2, n
        pair.check_kv(r, 2e-2)
    pair.close()


@pytest.mark.parametrize("n", [4, 5, 8, 9, 10])
@pytest.mark.parametrize("packed", [True, False], ids=["packed", "rowmajor"])
@pytest.mark.parametrize("name", ["k2048", "k768"])
def test_layouts_of_few_rows(name, packed, n):
    """Row counts on either side of where complete projections hold their rows row-major (up to four, nine) or in fragment
    order."""
    pair = Pair(SHAPES[name], 73, {0: 45}, flags=sp.SP_FLAG_PACKED_WEIGHTS if packed else 0)
    pair.insert(0, wl.tree_deep(73, n, 9))
    x = wl.hidden_rows(SHAPES[name], 73, ("layout", n), n)
    y, ref = pair.forward([0], [0], [n], x)
    assert rel_err(y - x, ref - x) <= 2e-2
    pair.check_kv(0, 2e-2)
    pair.close()
