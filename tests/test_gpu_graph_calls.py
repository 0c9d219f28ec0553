"""Calls of as many launches as are made one by one, and of more, which replay a graph of their own: the same bits as a stage that may
not replay (SP_FLAG_NO_GRAPHS), call after call."""
import pytest
import torch

import workloads as wl
import paper_2504_04104_amd as sp
from gpu_harness import Pair, to_dev

pytestmark = pytest.mark.gpu


# 21 rows of bf16: eight launches a layer; 6 rows: five; float32: five (nine with an attention cut into chunks, six)
@pytest.mark.parametrize("dtype,n_layers,n,prefix", [("bf16", 3, 21, 70), ("bf16", 4, 21, 70), ("bf16", 4, 6, 70), ("bf16", 5, 6, 600),
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
