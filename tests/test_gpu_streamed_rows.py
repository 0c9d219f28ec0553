"""The one-workgroup-per-CU kernel outside 49-160 rows of four column groups: row-major weights from one row on (whole lines
to LDS), 17-48 rows over weights in fragment order (two row tiles of gate/up: the eight-wave kernel without loading waves),
seven column groups (97-112 gate/up columns per CU), and a matrix
with more column tiles than CUs; against the CPU oracle."""
import numpy as np
import pytest

import workloads as wl
import paper_2504_04104_amd as sp
from gpu_harness import Pair, elementwise_figure, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,packed", [(1, False), (4, False), (5, False), (16, False), (17, False), (33, False), (48, False),
                                      (17, True), (32, True), (33, True), (48, True)])
def test_few_row_tiles(n, packed):
    """Two layers of the 8B stage's column counts over a short k range: up to 16 rows the second layer's gate/up takes the
    row's RMSNorm scale after the products."""
    check(wl.ModelShape(n_layers=2, d_model=512, n_q_heads=32, n_kv_heads=8, d_head=128, d_ff=14336), n, packed)


@pytest.mark.parametrize("n,packed", [(17, True), (48, True), (65, True), (128, True), (160, True), (1, False), (4, False), (5, False), (16, False), (17, False),
                                      (64, False), (96, False), (129, False), (160, False)])
def test_seven_column_groups(n, packed):
    check(wl.ModelShape(n_layers=1, d_model=512, n_q_heads=8, n_kv_heads=2, d_head=128, d_ff=28672), n, packed)


@pytest.mark.parametrize("n,packed", [(3, False), (17, False), (64, False), (100, False), (20, True), (100, True)])
def test_more_column_tiles_than_cus(n, packed):
    """QKV of 33792 columns: 264 tiles of 128, no k slices."""
    check(wl.ModelShape(n_layers=1, d_model=256, n_q_heads=256, n_kv_heads=4, d_head=128, d_ff=512), n, packed)


def check(shape, n, packed):
    """Increment y - x of small inputs element by element (2e-2 of the value plus 5e-2 of the rms a layer: about six tensors
    on the way are stored in bf16), cache rows at 2e-2 of the largest."""
    pair = Pair(shape, 61, {0: 21}, max_batch_nodes=160, flags=sp.SP_FLAG_PACKED_WEIGHTS if packed else 0)
    pair.insert(0, wl.tree_uniform_parents(61, n, 9, name=("streamed", n)))
    x = wl.hidden_rows(shape, 61, ("streamed", n), n) * np.float32(2.0 ** -6)
    y, ref = pair.forward([0], [0], [n], x)
    assert rel_err(y - x, ref - x) <= 2e-2
    assert elementwise_figure(y.astype(np.float64) - x, ref - x, 2e-2, 5e-2 * shape.n_layers) <= 1.0
    pair.check_kv(0, 2e-2)
    pair.close()
