"""Many rows over weights in fragment order: the 32 x 32 kernel at the row counts that select each of its heights, in gate/up
(the 8B stage's column counts over a short k range: d_ff = 14336 makes 112 column tiles, so that the rounds of workgroups
decide as they do at full depth) and in the plain products, whose write-out is another; one and two workgroups per CU, ragged
last tiles, several k slices; 161-192 rows of gate/up in the kernel of the fewer rows, 257-320 of a narrow one in blocks of
128.  Row-major weights stay in blocks of 128 and 256 rows."""
import os
import re

import numpy as np
import pytest

import workloads as wl
import paper_2504_04104_amd as sp
from gpu_harness import Pair, elementwise_figure, rel_err, to_dev, to_np

pytestmark = pytest.mark.gpu


# rows: 161 and 192 (twelve row tiles), 257 and 320 (160-row blocks), 321 and 384 (192), 400 (224), 512 (256), 513 and
# 639 (160, two per CU; the last tile of 639 one row short)
@pytest.mark.parametrize("rows,packed", [(161, True), (192, True), (192, False), (257, True), (320, True), (321, True), (384, True),
                                         (385, True), (400, True), (512, True), (513, True), (513, False), (639, True)])
def test_row_blocks(rows, packed):
    """Increment y - x of small inputs element by element (2e-2 of the value plus 5e-2 of the rms: about six tensors on
    the way are stored in bf16), cache rows at 2e-2 of the largest."""
    shape = wl.ModelShape(n_layers=1, d_model=512, n_q_heads=32, n_kv_heads=8, d_head=128, d_ff=14336)
    check(shape, rows, packed)


@pytest.mark.parametrize("rows", [385, 640, 700])
def test_k_slices_of_the_plain_products(rows):
    """K = 4096 in O and 3072 in the down projection with 512 to 768 columns: up to eight slices."""
    check(wl.ModelShape(n_layers=1, d_model=768, n_q_heads=32, n_kv_heads=4, d_head=128, d_ff=3072), rows, True)


def test_activations_longer_than_2_gb():
    """The most rows a call can carry (64 requests of 256 nodes) over d_ff = 66048: the products' rows take 2.16 GB, the
    last request's the part beyond 2^31 bytes.  Increment of its rows as above."""
    shape = wl.ModelShape(n_layers=1, d_model=256, n_q_heads=2, n_kv_heads=1, d_head=128, d_ff=66048)
    n_req, n = sp.SP_MAX_BATCH_REQ, sp.SP_MAX_TREE_NODES
    assert (n_req - 1) * n * shape.d_ff * 2 < 2 ** 31 < (n_req * n - 16) * shape.d_ff * 2
    pair = Pair(shape, 29, {r: 1 for r in range(n_req)}, max_batch_nodes=n_req * n, flags=sp.SP_FLAG_PACKED_WEIGHTS, oracle_reqs=[n_req - 1])
    trees = [wl.tree_uniform_parents(29, n, 9, name=("long", r)) for r in range(n_req)]
    pair.insert_batch(list(range(n_req)), trees)
    x = wl.hidden_rows(shape, 29, ("long",), n_req * n) * np.float32(2.0 ** -6)
    y = to_np(pair.gpu.stage_forward(list(range(n_req)), [0] * n_req, [n] * n_req, to_dev(x, pair.gpu)))[-n:]
    x = x[-n:]
    ref = pair.ora.stage_forward(n_req - 1, 0, x)
    assert rel_err(y - x, ref - x) <= 2e-2
    assert elementwise_figure(y.astype(np.float64) - x, ref - x, 2e-2, 5e-2) <= 1.0
    pair.close()


def wide_plan(rows, tiles, K, columns, cus=256, max_s=8):
    """The library's choice of (height in tiles of 32 rows, k slices) for a plain product, on the constants of its source."""
    src = open(os.path.join(os.path.dirname(sp.__file__), "csrc", "sp_gemm_wide.hip")).read()
    one, two = ([float(v) for v in re.search(name + r"\[\d\] = \{([^}]*)\}", src).group(1).split(",")] for name in ("one", "two"))
    best = None
    for rt in range(4, 9):
        for s in range(1, max_s + 1):
            n = -(-(-(-tiles // 8) * -(-rows // (rt * 32)) * s) // (cus // 8))
            loop = n // 2 * two[rt] + n % 2 * one[rt] if rt <= 5 else n * one[rt]
            us = loop * K / (4096 * s) + s * rows * columns * 4 / 1.95e6
            if best is None or us < best[0]:
                best = us, rt, s
    return best[1:]


# rows: height and slices of QKV (10240 columns, whose slices fill the scratch) and of O (8192 deep, 512 columns)
PLAIN = {513: ((4, 1), (5, 8)), 641: ((4, 1), (6, 8)), 767: ((4, 1), (6, 8)), 769: ((5, 1), (5, 6)), 850: ((5, 1), (7, 8)),
         895: ((5, 1), (7, 8)), 1000: ((6, 1), (8, 8)), 1023: ((6, 1), (8, 8))}


@pytest.mark.parametrize("rows", PLAIN)
def test_heights_of_the_plain_products(rows):
    """Heights of five to eight tiles with their write-out, last tiles of one row to one row short."""
    shape = wl.ModelShape(n_layers=1, d_model=512, n_q_heads=64, n_kv_heads=8, d_head=128, d_ff=512)
    assert (wide_plan(rows, 40, 512, 10240, max_s=1024 * 10240 // (rows * 10240)), wide_plan(rows, 2, 8192, 512)) == PLAIN[rows]
    check(shape, rows, True, max_rows=1024)


@pytest.mark.parametrize("rows", [257, 320, 321])
def test_gateup_in_one_round(rows):
    """64 column tiles, three row blocks: blocks of 128 rows up to 320."""
    check(wl.ModelShape(n_layers=1, d_model=512, n_q_heads=4, n_kv_heads=1, d_head=128, d_ff=8192), rows, True)


def check(shape, rows, packed, max_rows=704):
    n_req = (rows + 249) // 250
    counts = [rows // n_req + (r < rows % n_req) for r in range(n_req)]
    pair = Pair(shape, 29, {r: 19 + r for r in range(n_req)}, max_batch_nodes=max_rows, flags=sp.SP_FLAG_PACKED_WEIGHTS if packed else 0)
    for r, n in enumerate(counts):
        pair.insert(r, wl.tree_uniform_parents(29, n, 9, name=("many", rows, r)))
    x = wl.hidden_rows(shape, 29, ("many", rows), rows) * np.float32(2.0 ** -6)
    y, ref = pair.forward(list(range(n_req)), [0] * n_req, counts, x)
    assert rel_err(y - x, ref - x) <= 2e-2, rows
    assert elementwise_figure(y.astype(np.float64) - x, ref - x, 2e-2, 5e-2) <= 1.0, rows
    for r in range(n_req):
        pair.check_kv(r, 2e-2)
    pair.close()
