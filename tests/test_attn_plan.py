"""The split of a forward call's attention work (csrc/sp_plan.h, plain C++) on the CPU."""
import ctypes as C
import os
import random
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_04104_amd", "csrc")
DRIVER = """
#include <string.h>
#include "sp_plan.h"
extern "C" int split(int n, const int* rows, const int* spans, int n_q, int n_kv, int n_cu, long room, int* head, int* segs, AttnShape* shape) {
  AttnPlan p;
  memset(&p, 0, sizeof(p));
  p.n_seg = n;
  for (int i = 0; i < n; ++i) { p.seg_rows[i] = rows[i]; p.seg_P[i] = spans[i] - rows[i]; p.seg_T[i] = rows[i]; }
  if (!attn_split(p, n_q, n_kv, n_cu, (size_t)room)) return 0;
  const int h[] = {p.qt, p.total_items, p.any_split, p.units_total, p.loads};
  memcpy(head, h, sizeof(h));
  *shape = AttnShape(p);
  for (int i = 0; i < n; ++i) {
    const int s[] = {p.seg_item0[i], p.seg_chunks[i], p.seg_clen[i], p.seg_qblocks[i], p.seg_unit0[i]};
    memcpy(segs + i * 5, s, sizeof(s));
  }
  return 1;
}
extern "C" int shape_bytes() { return (int)sizeof(AttnShape); }
extern "C" int same_shape(const AttnShape* a, const AttnShape* b) { return *a == *b; }
"""
SHARED, STREAM, STREAM_REGS = 0, 1, 2


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "driver.cpp").write_text(DRIVER)
    so = str(d / "driver.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "driver.cpp"), "-o", so], check=True)
    lib = C.CDLL(so)

    def call(rows, spans, n_q=32, n_kv=8, n_cu=256, room=1 << 20):
        """Segments longest first, as the forward call enters them.  None where the partial results do not fit."""
        order = sorted(range(len(rows)), key=lambda i: -spans[i])
        r, s = ((C.c_int * len(rows))(*[v[i] for i in order]) for v in (rows, spans))
        head, segs, shape = (C.c_int * 5)(), (C.c_int * (5 * len(rows)))(), C.create_string_buffer(lib.shape_bytes())
        if not lib.split(len(rows), r, s, n_q, n_kv, n_cu, C.c_long(room), head, segs, shape):
            return None
        out = dict(zip(("qt", "items", "any_split", "units", "loads"), head))
        out["replays"] = lambda other: bool(lib.same_shape(shape, other["shape"]))
        out["shape"] = shape
        out["segs"] = np.array(segs).reshape(-1, 5)
        out["rows"], out["spans"] = list(r), list(s)
        return out
    return call


def test_every_plan_covers_its_ranges(split):
    """Chunks are whole tiles, none is empty, they cover the range; items and units of the segments follow each other; the
    partial results fit the room, and no call is refused (one chunk each needs none)."""
    r = random.Random(1)
    for _ in range(3000):
        n_kv = r.choice([1, 2, 4, 8])
        n_q = n_kv * r.choice([1, 2, 4, 8])
        rows = [r.choice([1, 2, 5, 9, 17, 64, 200]) for _ in range(r.choice([1, 1, 2, 5, 31, 64]))]
        spans = [v + int(2 ** r.uniform(0, 15)) for v in rows]
        room = r.choice([0, 2000, 1 << 20])
        p = split(rows, spans, n_q, n_kv, room=room)
        item, unit, any_split = 0, 0, 0
        for (item0, chunks, clen, qblocks, unit0), m, span in zip(p["segs"].tolist(), p["rows"], p["spans"]):
            assert clen % 32 == 0 and (chunks - 1) * clen < span <= chunks * clen
            assert qblocks == -(-m * (n_q // n_kv) // (16 * p["qt"]))
            assert (item0, unit0) == (item, unit)
            item += chunks * qblocks
            unit += chunks * m * n_q if chunks > 1 else 0
            any_split |= chunks > 1
        assert (item, unit, any_split) == (p["items"], p["units"], p["any_split"])
        assert unit <= room


# 32 query heads over 8 KV heads: a node is four query rows of a KV head
@pytest.mark.parametrize("rows,spans,n_q,qt", [
    # one request of more than 32 query rows, or half of them, among short ones: nearly as many blocks of 64 as of 32
    ([4] * 31 + [9], None, 32, 2), ([2] * 31 + [16], None, 32, 2), ([1, 9] * 16, None, 32, 2), ([4, 12] * 16, None, 32, 2),
    ([128] + [2] * 30, None, 32, 2), ([64] * 4 + [4] * 24, None, 32, 2), ([16] * 16 + [5] * 48, None, 32, 2),
    # half as many, but ranges of different lengths in one round of workgroups
    ([9] * 32, None, 32, 2), ([16] * 32, None, 32, 2), ([16] * 16, None, 64, 2),
    # ... in more than one
    ([16] * 40, None, 32, 4), ([25, 32] * 12, None, 32, 4), ([9, 12, 16, 8] * 12, None, 32, 4), ([32] * 16, None, 64, 4),
    # ranges of one length
    ([256], [2304], 64, 4), ([256], [2304], 32, 2),
    # small ones only
    ([8] * 64, None, 32, 2), ([4] * 64, None, 32, 1)])
def test_blocks_of_64_query_rows(split, rows, spans, n_q, qt):
    """... are taken where they are at most two thirds as many as blocks of 32, and a quarter more than the CUs or all of one request."""
    assert split(rows, spans or [700 + 97 * i % 3300 for i in range(len(rows))], n_q)["qt"] == qt


@pytest.mark.parametrize("rows,prefixes,cut", [
    # each request a block of its own: three rounds of tiles to save, four where the ranges occupy half of the CUs uncut
    ([1], [760], False), ([1], [780], True), ([1] * 5, [700] * 5, False), ([1] * 5, [1500] * 5, True), ([1] * 5, [1100] * 5, True),
    ([8] * 8, [1500] * 8, True), ([3] * 12, [1500] * 12, True), ([1] * 16, [1500] * 16, False), ([1] * 16, [2200] * 16, True),
    ([2] * 5, [700] * 4 + [1400], True),
    # blocks that share ranges: the more, the more rounds
    ([16], [900], False), ([16], [1200], True), ([37], [777], False), ([37], [1450], True), ([48], [1150], False), ([48], [1700], True),
    ([64], [1450], False), ([64], [2048], True), ([128], [2200], False), ([128], [2700], False), ([128], [3400], True),
    ([24] * 4, [1700] * 4, False), ([24] * 4, [3000] * 4, True)])
def test_ranges_whole_or_cut(split, rows, prefixes, cut):
    """Ranges of the 8B shape are cut into chunks only where the tiles that a wave saves are worth the merge."""
    assert bool(split(rows, [p + n for p, n in zip(prefixes, rows)])["any_split"]) == cut


def test_graphs_keep_to_their_kind_of_loads(split):
    """A graph holds the attention kernel that was launched when it was captured.  Calls of as many rows, blocks and chunks whose
    K/V rows come in another way have a graph of their own; other contexts, or the same requests in another order, do not."""
    two_blocks, one_each = split([8, 8, 8, 16], [700] * 4), split([8] * 5, [700] * 5)
    for name in ("qt", "items", "any_split", "units"):
        assert two_blocks[name] == one_each[name]
    assert (two_blocks["loads"], one_each["loads"]) == (SHARED, STREAM_REGS)
    assert not two_blocks["replays"](one_each)
    assert two_blocks["replays"](split([16, 8, 8, 8], [500, 600, 300, 64]))
    two_blocks, one_each = split([8, 8, 8, 16], [2000] * 4), split([8] * 5, [2000] * 5)
    assert two_blocks["units"] == one_each["units"] > 0
    assert (two_blocks["loads"], one_each["loads"]) == (SHARED, STREAM)
    assert not two_blocks["replays"](one_each)
    assert one_each["replays"](split([8] * 5, [1990, 1930, 1960, 2010, 1980]))
    assert split([8], [700])["loads"] == split([8], [5000])["loads"] == STREAM
    assert split([64], [5000])["loads"] == SHARED
