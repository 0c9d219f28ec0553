"""49-160 rows: the kernels with two strips of weight rows per wave, at the edges of their row tiles, against the CPU
oracle.  The shape has the 8B stage's column counts (QKV 6144 columns: 96-column tiles; d_ff = 14336 and 16384: 56 and 64
gate/up columns per CU, with a short and a full last column group) over a short k range."""
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
    pair = Pair(shape, 83, {0: 21}, max_batch_nodes=192, flags=sp.SP_FLAG_PACKED_WEIGHTS if packed else 0)
    pair.insert(0, wl.tree_uniform_parents(83, n, 9, name=("mid", n)))
    x = wl.hidden_rows(shape, 83, ("mid", n), n) * np.float32(2.0 ** -6)
    y, ref = pair.forward([0], [0], [n], x)
    assert rel_err(y - x, ref - x) <= 2e-2
    assert elementwise_figure(y.astype(np.float64) - x, ref - x, 2e-2, 5e-2) <= 1.0
    pair.check_kv(0, 2e-2)
    pair.close()
