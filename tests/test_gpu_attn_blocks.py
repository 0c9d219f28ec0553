"""Attention of many requests at once: blocks of 64 query rows whose tiles two waves share, blocks of 32, and ranges streamed through
registers, at context lengths around the edges of tiles and runs, against the CPU oracle.  The requests' contexts are in no
order, so that the longest-first order of the work differs from the call's."""
import numpy as np
import pytest

import workloads as wl
import paper_2504_04104_amd as sp
from gpu_harness import Pair, elementwise_figure, rel_err

pytestmark = pytest.mark.gpu

SHAPE = wl.ModelShape(n_layers=1, d_model=512, n_q_heads=32, n_kv_heads=8, d_head=128, d_ff=512)
CONTEXTS = [33, 1, 257, 31, 128, 513, 32, 127, 300, 64, 5, 129, 255, 63, 96, 256, 224, 2, 192, 65, 160, 97, 385, 17]


@pytest.mark.parametrize("page_slots", [0, 32], ids=["contiguous", "pages32"])
@pytest.mark.parametrize("rows", [
    # one to three blocks of 64 query rows (four per node), 43 in all: 344 workgroups
    pytest.param([33, 16, 17, 1, 32, 31, 48, 8, 33, 16, 17, 4, 32, 31, 2, 9, 33, 16, 17, 1, 32, 31, 40, 8], id="blocks_of_64"),
    # 31 blocks of 64: blocks of 32
    pytest.param([17] * 7 + [16] * 17, id="blocks_of_32"),
    # a single block each: 24 streamed ranges, one and two query tiles
    pytest.param([8, 1, 3, 5, 8, 2] * 4, id="streamed"),
    pytest.param([4, 1, 3, 2, 4, 2] * 4, id="streamed_one_tile")])
def test_ragged_contexts(rows, page_slots):
    """Increment y - x of small inputs element by element (2e-2 of the value plus 5e-2 of the rms: about six tensors on the way
    are stored in bf16), twice with other rows, then the cache rows."""
    n = len(rows)
    pair = Pair(SHAPE, 91, dict(enumerate(CONTEXTS)), max_batch_nodes=640, page_slots=page_slots, norm1_gain=4.0)
    pair.insert_batch(list(range(n)), [wl.tree_deep(91 + q, r, 9) for q, r in enumerate(rows)])
    for k in range(2):
        x = wl.hidden_rows(SHAPE, 91, ("blocks", k), sum(rows)) * np.float32(2.0 ** -6)
        y, ref = pair.forward(list(range(n)), [0] * n, rows, x)
        assert rel_err(y - x, ref - x) <= 2e-2, k
        assert elementwise_figure(y.astype(np.float64) - x, ref - x, 2e-2, 5e-2) <= 1.0, k
    for q in range(n):
        pair.check_kv(q, 2e-2)
    pair.close()


@pytest.mark.parametrize("n", [33, 3])
def test_requests_that_take_pages_at_once(n):
    """More requests than an insert launch carries pages for (and a few) whose rows reach a new page, one of them three, twice: the
    cache rows land there and the attention finds them."""
    pair = Pair(SHAPE, 93, {q: 31 + q % 2 for q in range(n)}, max_batch_nodes=640, page_slots=32)
    for k in range(2):
        rows = [70 if q == 1 and k == 0 else 5 for q in range(n)]
        first = pair.insert_batch(list(range(n)), [wl.tree_deep(93 + q, r, 9) for q, r in enumerate(rows)])
        x = wl.hidden_rows(SHAPE, 93, ("pages", k), sum(rows))
        y, ref = pair.forward(list(range(n)), first, rows, x)
        assert rel_err(y - x, ref - x) <= 2e-2, k
        for q in range(n):
            pair.check_kv(q, 2e-2)
        if k == 0:
            for q in range(n):
                pair.prune(q, sp.SP_CLEAR, 0)
    pair.close()


@pytest.mark.parametrize("n,prefixes", [(2, [571, 766, 767]), (5, [571, 1019, 1020]), (20, [1004, 1005, 1532, 1790])],
                         ids=["one_block", "two_blocks", "five_blocks"])
def test_one_chunk_or_several(n, prefixes):
    """One request whose cache range (with its n nodes) lies on either side of where it is cut into chunks: four rounds of 256 slots
    where it is a single block of query rows, five where it is a few that share it."""
    shape = wl.ModelShape(n_layers=1, d_model=512, n_q_heads=64, n_kv_heads=8, d_head=128, d_ff=512)
    for P in prefixes:
        pair = Pair(shape, 95, {0: P}, norm1_gain=4.0)
        pair.insert(0, wl.tree_deep(95, n, 7))
        x = wl.hidden_rows(shape, 95, ("chunks", P), n) * np.float32(2.0 ** -6)
        y, ref = pair.forward([0], [0], [n], x)
        assert rel_err(y - x, ref - x) <= 2e-2, P
        assert elementwise_figure(y.astype(np.float64) - x, ref - x, 2e-2, 5e-2) <= 1.0, P
        pair.close()
