"""49-160 rows: the kernel with two strips of weight rows per wave and loading waves, at the edges of its row tiles and of
its k loops, and what runs beside it, against the CPU oracle.  The first shape has the 8B stage's column counts (QKV 6144 columns: 96-column tiles; d_ff = 14336 and 16384: 56
and 64 gate/up columns per CU, with a short and a full last column group) over a short k range."""
import numpy as np
import pytest

import workloads as wl
import paper_2504_04104_amd as sp
from gpu_harness import Pair, elementwise_figure, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d_ff,packed", [(49, 14336, True), (64, 16384, False), (65, 14336, False), (81, 14336, True),
                                           (96, 16384, True), (97, 14336, True), (128, 14336, False), (129, 14336, True),
                                           (145, 16384, False), (160, 14336, True), (161, 14336, True)])
def test_row_tiles(n, d_ff, packed):
    """Increment y - x of small inputs element by element (2e-2 of the value plus 5e-2 of the rms: about six tensors on
    the way are stored in bf16), cache rows at 2e-2 of the largest."""
    shape = wl.ModelShape(n_layers=1, d_model=512, n_q_heads=32, n_kv_heads=8, d_head=128, d_ff=d_ff)
    check_increment(shape, [n], packed)


# Products and gate/up whose workgroups walk eight to sixteen chunks of 128 k, the ring of panels and weight sets several
# times round and left at each of its places, at each number of row tiles; row-major gate/up from staggered starts.
@pytest.mark.parametrize("n,d_model,d_ff,packed", [(64, 1024, 14336, True), (64, 1280, 16384, False), (96, 1536, 14336, False),
                                                   (96, 1280, 14336, True), (128, 2048, 16384, False), (128, 1792, 14336, True),
                                                   (145, 1024, 14336, False), (160, 2048, 14336, True)])
def test_long_k_ranges(n, d_model, d_ff, packed):
    check_increment(wl.ModelShape(n_layers=1, d_model=d_model, n_q_heads=8, n_kv_heads=2, d_head=128, d_ff=d_ff), [n], packed)


@pytest.mark.parametrize("packed", [True, False], ids=["packed", "rowmajor"])
def test_96_column_tiles_of_resident_weights(packed):
    """O with 3072 columns: tiles of 96, its weights read with ordinary loads."""
    check_increment(wl.ModelShape(n_layers=1, d_model=3072, n_q_heads=8, n_kv_heads=2, d_head=128, d_ff=512), [65, 96, 145], packed)


def test_two_strips_per_wave_of_a_wide_matrix():
    """97-128 rows of a matrix that leaves its workgroups two k slices (11264 columns, 6144 deep: 88 tiles of 128
    columns on 256 CUs).  The element-wise allowance is 7.5e-2 of the rms here: the plain kernels, whose float32
    sums run in another order, need 6.0e-2 on the same inputs (1.2 million numbers a call)."""
    shape = wl.ModelShape(n_layers=1, d_model=11264, n_q_heads=16, n_kv_heads=2, d_head=128, d_ff=6144)
    weights = wl.layer_weights(shape, 83, 0)
    for packed in (True, False):
        check_increment(shape, [97, 128], packed, atol_rms=7.5e-2, weights=lambda l: weights)


def check_increment(shape, rows, packed, atol_rms=5e-2, **kw):
    pair = Pair(shape, 83, {r: 21 for r in range(len(rows))}, max_batch_nodes=192, flags=sp.SP_FLAG_PACKED_WEIGHTS if packed else 0, **kw)
    for r, n in enumerate(rows):
        pair.insert(r, wl.tree_uniform_parents(83, n, 9, name=("mid", n)))
        x = wl.hidden_rows(shape, 83, ("mid", n), n) * np.float32(2.0 ** -6)
        y, ref = pair.forward([r], [0], [n], x)
        assert rel_err(y - x, ref - x) <= 2e-2, n
        assert elementwise_figure(y.astype(np.float64) - x, ref - x, 2e-2, atol_rms) <= 1.0, n
        pair.check_kv(r, 2e-2)
    pair.close()
