"""Verification kernels on logits that are known exactly: the vocabulary matrix has one non-zero per row and the roots'
rows are all ones, so that a logit is that one number (RMSNorm of ones is 1 in bf16).  The choices can then be compared
without a margin: tile statistics of the logits (64- and 128-column tiles), rows full of ties, rows that one token
rules, candidate groups of every size."""
import numpy as np
import pytest
import torch

import workloads as wl
import paper_2504_04104_amd as sp
from gpu_harness import Pair
from oracle.verify import sample_token, sampling_candidates

pytestmark = pytest.mark.gpu

SHAPE = wl.ModelShape(n_layers=1, d_model=512, n_q_heads=4, n_kv_heads=2, d_head=128, d_ff=768)


def exact_head(logits, packed):
    V = len(logits)
    w = torch.zeros(V, SHAPE.d_model)
    w[torch.arange(V), torch.arange(V) % SHAPE.d_model] = torch.from_numpy(logits.astype(np.float32))
    w = w.to("cuda:0", torch.bfloat16)
    return {"norm": torch.ones(SHAPE.d_model, dtype=torch.bfloat16, device="cuda:0"), "wvocab": sp.pack_matrix(w) if packed else w}


def draw_logits(kind, V, seed):
    r = np.random.RandomState(seed)
    l = r.normal(0.0, 2.0, V)
    if kind == "peaked":
        l[r.randint(V)] = 14.0
    if kind == "levels":                  # more tied tokens than the short candidate list holds
        l = r.choice([-1.0, 0.5, 2.0], V)
    return torch.from_numpy(l).to(torch.bfloat16).double().numpy()


@pytest.mark.parametrize("kind", ["spread", "peaked", "levels"])
@pytest.mark.parametrize("n,V,packed", [(1, 64 * 140, True), (1, 64 * 140, False), (17, 128 * 100, True), (33, 64 * 141, False),
                                        (64, 128 * 80, True), (3, 64 * 79, True)])
def test_sampling_from_exact_logits(n, V, packed, kind):
    """The token drawn at the middle of a candidate's interval is that candidate (64 * 79 columns: too few tiles for the
    bound at 80 candidates, the kernel walks the row)."""
    logits = draw_logits(kind, V, V + n)
    pair = Pair(SHAPE, 5, {r: 9 for r in range(n)}, max_batch_nodes=64, oracle=False, flags=sp.SP_FLAG_PACKED_WEIGHTS if packed else 0)
    head = exact_head(logits, packed)
    x = torch.ones(n, SHAPE.d_model, dtype=torch.bfloat16, device="cuda:0")
    r = np.random.RandomState(n)
    for T, p, k in ((0.6, 0.9, 80), (1.0, 1.0, 7), (0.3, 0.999, 80)):
        toks, ps = sampling_candidates(logits, T, p, k)
        c = np.concatenate(([0.0], np.cumsum(ps))) / np.sum(ps)
        wide = [j for j in range(len(ps)) if c[j + 1] - c[j] > 1e-4]
        picks = [wide[0], wide[-1]][:n] + [wide[r.randint(len(wide))] for _ in range(n - 2)]
        u = [float(np.float32(0.5 * (c[j] + c[j + 1]))) for j in picks]
        got = pair.gpu.verify_sample(head, list(range(n)), x, T, p, k, u)
        for (node, tok), j, v in zip(got, picks, u):
            assert sample_token(logits, T, p, k, v) == toks[j]
            assert tok == toks[j] and node == -1, (T, p, k, j)
    pair.close()


@pytest.mark.parametrize("V", [64 * 255, 128 * 127])
def test_sampling_without_room_for_statistics(V):
    """64 rows of logits in tiles of 64 and of 128 columns that fill the workspace so far that the tiles' statistics do not
    fit behind them: the row is walked tile by tile."""
    test_sampling_from_exact_logits(64, V, True, "spread")


@pytest.mark.parametrize("n_child", [1, 2, 15, 16, 17, 27, 32, 33, 63, 64, 65, 128, 129, 200])
@pytest.mark.parametrize("n,V", [(1, 5003), (2, 64 * 140), (40, 64 * 70)])
def test_lossy_from_exact_logits(n, V, n_child):
    """Relaxed: the child whose token has the highest logit, the first among equals.  Top-p: of the children whose token
    has less than top_p of the mass in front of it, the one with the highest draft probability (a child within 1e-5 of
    top_p is not asked for)."""
    flags = 0
    logits = draw_logits("spread", V, V + n_child)
    head = exact_head(logits, False)
    pair = Pair(SHAPE, 5, {r: 9 for r in range(n)}, max_batch_nodes=64, oracle=False, flags=flags)
    x = torch.ones(n, SHAPE.d_model, dtype=torch.bfloat16, device="cuda:0")
    order = np.lexsort((np.arange(V), -logits))
    prob = np.exp(logits - logits.max())
    before = np.empty(V)
    before[order] = np.concatenate(([0.0], np.cumsum(prob[order])))[:-1] / prob.sum()
    r = np.random.RandomState(V + n)
    kids = []
    for q in range(n):
        tok = [int(order[r.randint(min(V, 3000))]) for _ in range(n_child)]
        tok = [t if abs(before[t] - 0.9) > 1e-5 else -1 for t in tok]
        if n_child > 2:
            tok[1] = V + 5                 # outside the vocabulary
        draft = [float(np.float32(v)) for v in r.choice([0.125, 0.25, 0.5], n_child)]
        pair.gpu.tree_insert(q, [-1] * n_child, tok, draft)
        kids.append((tok, draft))
    relaxed = pair.gpu.verify_lossy(head, list(range(n)), x, sp.SP_VERIFY_RELAXED)
    top_p = pair.gpu.verify_lossy(head, list(range(n)), x, sp.SP_VERIFY_TOP_P, 0.9)
    for q, (tok, draft) in enumerate(kids):
        ok = [i for i, t in enumerate(tok) if 0 <= t < V]
        want = max(ok, key=lambda i: (logits[tok[i]], -i)) if ok else -1
        assert relaxed[q] == (want, int(order[0]))
        ok = [i for i in ok if before[tok[i]] < 0.9]
        want = max(ok, key=lambda i: (draft[i], -i)) if ok else -1
        assert top_p[q] == (want, int(order[0])), q
    pair.close()


@pytest.mark.parametrize("n_child", [3, 16, 17, 32, 33, 64, 100, 200])
@pytest.mark.parametrize("tie", [0.0, 1.5])
@pytest.mark.parametrize("n,V", [(1, 5003), (2, 64 * 140), (40, 64 * 70)])
def test_lossy_among_equal_tokens(n, V, tie, n_child):
    """Most tokens have the same logit (zero: the next float below is a denormal), in runs that fill slices; some stand above, some
    have no mass.  A child's mass is counted in tied tokens; the children, tokens all over the row, have draft probabilities that
    grow with it, and top_p lies half a token behind or in front of one child's: a single tied token miscounted changes the
    verdict (float32 sums of 9000 terms are off by less than a hundredth of one)."""
    r = np.random.RandomState(V + n_child)
    logits = np.full(V, tie)
    for value, count in ((tie + 2.0, 12), (-120.0, V // 12), (-np.inf, V // 12)):
        logits[r.choice(V, count, replace=False)] = value
    at = int(r.randint(V // 2))
    logits[at:at + 2100] = tie
    pair = Pair(SHAPE, 5, {q: 9 for q in range(n)}, max_batch_nodes=64, oracle=False)
    x = torch.ones(n, SHAPE.d_model, dtype=torch.bfloat16, device="cuda:0")
    head = exact_head(logits, False)
    mass = np.exp(logits - tie)
    order = np.lexsort((np.arange(V), -logits))
    before = np.empty(V)
    before[order] = np.concatenate(([0.0], np.cumsum(mass[order])))[:-1]
    tied = np.flatnonzero(logits == tie)
    kids = []
    for q in range(n):
        tok = np.sort(r.choice(tied[1:], n_child - 1, replace=False))
        tok = [int(tied[0])] + [int(t) for t in tok]        # ascending: each has more in front of it
        draft = [float(np.float32((k + 1) / (n_child + 1))) for k in range(n_child)]
        mix = r.permutation(n_child)
        kids.append([tok[k] for k in mix])
        pair.gpu.tree_insert(q, [-1] * n_child, kids[q], [draft[k] for k in mix])
    for j in sorted({0, 1, n_child // 2, n_child - 1} | set(r.randint(0, n_child, 4))):
        for half in (0.5, -0.5):
            q0 = int(r.randint(n))
            bound = before[sorted(kids[q0])[j]] + half
            got = pair.gpu.verify_lossy(head, list(range(n)), x, sp.SP_VERIFY_TOP_P, float(bound / mass.sum()))
            for q in range(n):
                if q != q0 and min(abs(before[t] - bound) for t in kids[q]) < 0.25:
                    continue
                ok = [t for t in kids[q] if before[t] < bound]
                want = kids[q].index(max(ok)) if ok else -1
                assert got[q] == (want, int(order[0])), (q, j, half)
    pair.close()


@pytest.mark.parametrize("V,first_masked", [(64 * 140, 8448), (5003, 4608)])
def test_lossy_with_masked_tail(V, first_masked):
    """The end of the vocabulary masked with minus infinity, as padding rows are: a slice of tokens that holds nothing
    else has no mass, and neither rule may notice it."""
    logits = draw_logits("spread", V, V)
    logits[first_masked:] = -np.inf
    head = exact_head(logits, False)
    pair = Pair(SHAPE, 5, {0: 9}, max_batch_nodes=64, oracle=False)
    x = torch.ones(1, SHAPE.d_model, dtype=torch.bfloat16, device="cuda:0")
    order = np.lexsort((np.arange(V), -logits))
    tok = [int(order[2000]), int(order[40]), V - 1, int(order[0])]
    draft = [0.5, 0.25, 0.75, 0.125]
    pair.gpu.tree_insert(0, [-1] * 4, tok, draft)
    assert pair.gpu.verify_lossy(head, [0], x, sp.SP_VERIFY_RELAXED) == [(3, tok[3])]
    mass = np.cumsum(np.exp(logits[order] - logits.max()))
    assert mass[39] / mass[-1] < 0.9 < mass[1999] / mass[-1]
    assert pair.gpu.verify_lossy(head, [0], x, sp.SP_VERIFY_TOP_P, 0.9) == [(1, tok[3])]
    pair.close()


def test_sampling_never_draws_a_token_without_probability():
    """A few tokens hold all the mass (the others' exponentials are zero in float32) and u is the largest number below
    one: the draw is the last token with a probability, whatever the rounding of the running sums."""
    V, u = 64 * 140, float(np.float32(1.0) - np.float32(2.0 ** -24))
    pair = Pair(SHAPE, 5, {0: 9}, max_batch_nodes=64, oracle=False)
    x = torch.ones(1, SHAPE.d_model, dtype=torch.bfloat16, device="cuda:0")
    r = np.random.RandomState(3)
    wrong = []
    for case in range(60):
        k = 3 + case % 12
        logits = np.full(V, -120.0)
        top = r.choice(V, k, replace=False)
        logits[top] = 1.0 + r.randint(0, 16, k) / 8.0
        last = int(np.lexsort((np.arange(V), -logits))[k - 1])
        (_, tok), = pair.gpu.verify_sample(exact_head(logits, False), [0], x, 1.0, 1.0, 80, [u])
        if tok != last:
            wrong.append((case, k, float(logits[tok])))
    pair.close()
    assert not wrong, wrong


@pytest.mark.parametrize("packed", [True, False], ids=["packed", "rowmajor"])
@pytest.mark.parametrize("n,V", [(1, 704), (3, 640), (4, 704), (5, 640), (8, 704), (9, 640), (16, 640), (17, 704), (17, 640), (33, 640), (48, 704),
                                 (48, 640), (64, 640), (70, 704)])
def test_vocabulary_products_of_distinct_rows(n, V, packed):
    """Output head, relaxed and top-p verification of rows that all differ, tiles of 64 and of 128 columns, one to eight row
    tiles and the ends of their blocks: tokens and winning logits within 2e-2 of the largest logit (rows and weights are
    stored in bf16), as everywhere."""
    reqs = list(range(min(n, 64)))
    pair = Pair(SHAPE, 37, {r: 5 + r % 7 for r in reqs}, max_batch_nodes=80, vocab=V, flags=sp.SP_FLAG_PACKED_WEIGHTS if packed else 0)
    counts = [n - len(reqs) + 1] + [1] * (len(reqs) - 1)
    for r, c in zip(reqs, counts):
        pair.insert(r, [-1] * c, [(r * 31 + 7 * k) % V for k in range(c)], [0.5] * c)
    x = torch.from_numpy(wl.hidden_rows(SHAPE, 37, ("head", n), n)).to("cuda:0", torch.bfloat16)
    pair.gpu.stage_forward(reqs, [0] * len(reqs), counts, x)
    for r, c in zip(reqs, counts):
        pair.ora.stage_forward(r, 0, np.zeros((c, SHAPE.d_model)))
    pair.verify_head(reqs, [0] * len(reqs), counts, x, 2e-2)
    rows = x[:len(reqs)].contiguous()
    for mode in ("relaxed", "top_p"):
        pair.verify_lossy(reqs, rows, mode, 0.9, 2e-2)
    pair.close()
