"""Calls of as many launches as are made one by one (24), and of more, which replay a graph of their own: the same bits as a stage that
may not replay (SP_FLAG_NO_GRAPHS), call after call."""
import random

import pytest
import torch

import workloads as wl
import paper_2504_04104_amd as sp
from gpu_harness import Pair, to_dev, use_own_stream

pytestmark = pytest.mark.gpu


# 21 rows of bf16: eight launches a layer; 6 rows: five (six with an attention cut into chunks); float32: five
@pytest.mark.parametrize("dtype,n_layers,n,prefix", [("bf16", 3, 21, 70), ("bf16", 4, 21, 70), ("bf16", 4, 6, 70), ("bf16", 5, 6, 1300),
                                                     ("f32", 4, 6, 70), ("f32", 5, 6, 70)])
def test_replayed_calls(dtype, n_layers, n, prefix):
    shape = wl.ModelShape(n_layers=n_layers, d_model=512, n_q_heads=4, n_kv_heads=2, d_head=128, d_ff=768, dtype=dtype)
    flags = sp.SP_FLAG_PACKED_WEIGHTS if dtype == "bf16" else 0
    a = Pair(shape, 28, {0: prefix}, flags=flags, oracle=False)
    b = Pair(shape, 28, {0: prefix}, flags=flags | sp.SP_FLAG_NO_GRAPHS, oracle=False)
    par = wl.tree_uniform_parents(28, n, 5, name=("r",))
    for rep in range(5):
        outs = []
        for pair in (a, b):
            g = pair.gpu
            g.request_init(0, pair.base[0], pair.cap[0], prefix)
            g.tree_insert(0, par)
            y = g.stage_forward([0], [0], [n], to_dev(wl.hidden_rows(shape, 28, ("r", rep), n), g))
            g.tree_prune(0, sp.SP_DROP, 2)
            g.kv_compact(0)
            outs.append((y.clone(), pair.rows(0, 0, prefix + 2)))
        torch.cuda.synchronize()
        for u, v in zip(outs[0], outs[1]):
            assert torch.equal(u, v), rep
    a.close()
    b.close()


ROWS_64 = [33, 16, 17, 1, 32, 31, 48, 8, 33, 16, 17, 4, 32, 31, 2, 9, 33, 16, 17, 1, 32, 31, 40, 8]
PLANS = {   # layers, query and KV heads, rows of a call's requests, their contexts (in any order the same blocks and chunks)
    "one_block_each": (6, 8, 2, [4, 1, 3, 2, 4, 2], [33, 1, 257, 31, 128, 300]),
    "one_block_each_cut": (6, 8, 2, [3, 2, 4], [1040, 1100, 1222]),
    "one_request": (6, 8, 2, [6], [300]),
    "shared_blocks": (4, 8, 2, [9, 12, 5, 20], [33, 130, 257, 64]),
    "shared_blocks_cut": (4, 8, 2, [9, 12], [2080, 2222]),
    "blocks_of_64": (4, 32, 8, ROWS_64, [33 + 29 * i % 200 for i in range(24)]),
    "f32": (6, 4, 4, [5, 1, 9], [33, 130, 64])}


@pytest.mark.parametrize("page_slots", [0, 32], ids=["contiguous", "pages32"])
@pytest.mark.parametrize("name", PLANS)
def test_one_graph_under_changing_plans(name, page_slots):
    """Calls of one shape (30 launches and more) again and again, each with other requests in another order, other contexts, first
    nodes, input rows and result tensors, every third in place; a call of another shape and the set-up of all requests stand
    between them.  A call writes its result, the new cache rows and nothing else."""
    n_layers, n_q, n_kv, rows, contexts = PLANS[name]
    shape = wl.ModelShape(n_layers=n_layers, d_model=512, n_q_heads=n_q, n_kv_heads=n_kv, d_head=64 if name == "f32" else 128, d_ff=512,
                          dtype="f32" if name == "f32" else "bf16")
    use_own_stream()
    r = random.Random(31)
    tree = max(rows) + 3
    ids = list(range(len(rows)))
    cap = -(-(max(contexts) + tree) // 32) * 32
    layers = [sp.pack_layer_weights(wl.layer_weights(shape, 31, l), shape.dtype) for l in range(n_layers)]
    flags = sp.SP_FLAG_PAGED_KV if page_slots else 0
    if shape.dtype == "bf16":
        layers, flags = sp.pack_weights(shape, layers), flags | sp.SP_FLAG_PACKED_WEIGHTS
    stages = [sp.Stage(shape, layers, kv_slots=cap * len(rows), max_requests=len(rows), max_batch_nodes=tree * len(rows), flags=f,
                       page_slots=page_slots) for f in (flags, flags | sp.SP_FLAG_NO_GRAPHS)]
    stages[0].kv_view().normal_()
    stages[1].kv.copy_(stages[0].kv)
    parents = [wl.tree_deep(31 + q, tree, 9) for q in ids]
    results = []
    for rep in range(7):
        calls, lengths, first = r.sample(ids, len(ids)), r.sample(contexts, len(ids)), [r.randint(0, tree - n) for n in rows]
        x_all = to_dev(wl.hidden_rows(shape, 31, ("all", rep), tree * len(rows)), stages[0])
        x = to_dev(wl.hidden_rows(shape, 31, ("rows", rep), sum(rows)), stages[0])
        ys = []
        for st in stages:
            for q in ids:
                st.request_init(q, 0 if page_slots else cap * q, cap, lengths[q])
            st.tree_insert_batch(ids, parents)
            st.stage_forward(ids, [0] * len(ids), [tree] * len(ids), x_all)
            xs = x.clone()
            y = xs if rep % 3 == 2 else torch.full_like(x, float("nan"))
            st.stage_forward(calls, first, rows, xs, y)
            ys.append(y)
        assert bool(torch.isfinite(ys[1]).all())
        assert torch.equal(ys[0], ys[1]), rep
        assert torch.equal(stages[0].kv, stages[1].kv), rep
        results.append((ys[0], ys[1].clone()))
    for y, want in results:
        assert torch.equal(y, want)
    for st in stages:
        st.close()
