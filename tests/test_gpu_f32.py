"""float32 kernels at the edges of their tiles against the CPU oracle: k ranges that end inside a step of sixteen, columns
that end inside a tile, one to four row tiles per workgroup, both head sizes, contexts shorter than the four waves'
shares."""
from dataclasses import replace

import numpy as np
import pytest
import torch

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
    argument, on trees whose last levels have ancestors all over the range.  Three calls of five layers (25 launches): the
    later ones replay a graph."""
    shape = replace(shape, n_layers=5)
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


@pytest.mark.parametrize("n", [1, 16, 33, 65])
@pytest.mark.parametrize("shape", SHAPES.values(), ids=SHAPES.keys())
def test_f32_rows_of_any_scale(shape, n):
    """Rows from 2^-12 to 2^12 of the usual size in one call: each takes its own RMSNorm scale after the products.  A row's
    increment within 2e-5 of its largest value (as above) plus the roundings of x + increment, two additions a layer at
    half a unit of 2^-23 of the row's largest value, doubled."""
    pair = Pair(shape, 29, {0: 37}, max_batch_nodes=80)
    pair.insert(0, wl.tree_deep(29, n, 20))
    scale = np.float32(2.0) ** ((np.arange(n) * 7) % 25 - 12).astype(np.float32)
    x = wl.hidden_rows(shape, 29, ("f32 scales", n), n) * scale[:, None]
    y, ref = pair.forward([0], [0], [n], x)
    pair.close()
    err = np.abs((y - x) - (ref - x)).max(1)
    assert (err <= 2e-5 * np.abs(ref - x).max(1) + 4 * 2.0 ** -23 * np.abs(ref).max(1)).all()


@pytest.mark.parametrize("page_slots", [0, 32], ids=["contiguous", "pages32"])
@pytest.mark.parametrize("shape", SHAPES.values(), ids=SHAPES.keys())
def test_f32_infinite_value_row(shape, page_slots):
    """An infinity in the committed context's first V row makes that column of the head's attention rows infinite and
    leaves the other columns finite: slots that a row does not see (siblings, the padding of a step) add nothing.  Read
    where the kernel leaves the rows, in the workspace (behind the row descriptors, the rotary tables, the residual rows,
    the normalised rows and the queries, each part aligned to 256 bytes); past the norm that follows all would be NaN."""
    n, MB, col = 5, 16, 3
    pair = Pair(shape, 29, {0: 41}, max_batch_nodes=MB, page_slots=page_slots, oracle=False)
    g = pair.gpu
    first = int(g.logical_slots(0, 0, 1)[0]) if page_slots else pair.base[0]
    g.kv_view()[shape.n_layers - 1, 1, 0, first, col] = float("inf")
    g.tree_insert(0, [-1] * n)
    x = torch.from_numpy(wl.hidden_rows(shape, 29, ("inf",), n)).to("cuda:0")
    g.stage_forward([0], [0], [n], x)
    dq = shape.n_q_heads * shape.d_head
    parts = (MB * 32, MB * shape.d_head * 4, MB * shape.d_model * 4, MB * shape.d_model * 4, MB * dq * 4)
    at = sum((b + 255) // 256 * 256 for b in parts)
    rows = g.workspace[at:at + n * dq * 4].view(torch.float32).view(n, shape.n_q_heads, shape.d_head).cpu()
    pair.close()
    want_inf = torch.zeros_like(rows, dtype=torch.bool)
    want_inf[:, :shape.n_q_heads // shape.n_kv_heads, col] = True
    assert int((~torch.isposinf(rows[want_inf])).sum()) == 0
    assert int((~torch.isfinite(rows[~want_inf])).sum()) == 0


@pytest.mark.parametrize("page_slots", [0, 32], ids=["contiguous", "pages32"])
@pytest.mark.parametrize("n", [128, 129, 250])
def test_f32_many_qkv_workgroups(n, page_slots):
    """6144 QKV columns: up to 128 rows norm and rotation join the product, from 129 on they are launches of their own
    (bound as in test_f32_tiles)."""
    shape = wl.ModelShape(n_layers=5, d_model=72, n_q_heads=16, n_kv_heads=16, d_head=128, d_ff=40, rms_eps=1e-6, dtype="f32")
    pair = Pair(shape, 29, {0: 61}, max_batch_nodes=256, page_slots=page_slots)
    pair.insert(0, wl.tree_deep(29, n, 20))
    pair.gpu.profile_begin(11, 16)               # SP_K_ROPE_KV
    for k in range(3):
        x = wl.hidden_rows(shape, 29, ("f32 many", n, k), n)
        y, ref = pair.forward([0], [0], [n], x)
        assert rel_err(y - x, ref - x) <= 2e-5
    assert (pair.gpu.profile_end()[0] > 0) == (n > 128)
    x = wl.hidden_rows(shape, 29, ("f32 many", n), n)
    for k in range(3):                            # 25 launches and more: replayed from the second or third on
        y, ref = pair.forward([0], [0], [n], x)
        assert rel_err(y - x, ref - x) <= 2e-5
    pair.check_kv(0, 2e-5)
    pair.close()
