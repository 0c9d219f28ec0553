"""The calls that users of the stage library make, as cases that can be timed and compared.

A case is a dict of plain values; `prepare` builds what a serving program holds before the call (weights, cache,
request, schedule), `run` is one pass through the public entry points, `exact` the same pass in float64 with plain
torch.  The kinds:

  tree    one pipeline step of one request: reset to the committed context, insert a tree, forward its nodes, accept
          a child of the root, compact the cache and the rows in flight
  stream  the same request fed a few nodes at a time: insert, forward, prune, compact, several steps in a row
  batch   dynamic batching: clear, insert, forward over many requests; `steady` drops a subtree per request, compacts
          and feeds a second, small level
  head    output head of the last stage: the top-1 token of every row
  verify  top-p or stochastic verification of the root's successor, one row of logits per request
  grow    fixed-width expansion of the tree bottom and the insert of the level it gives
"""
from __future__ import annotations

import math
import random
from dataclasses import dataclass

import numpy as np
import torch

import paper_2504_04104_amd as sp

DEV = "cuda:0"


@dataclass(frozen=True)
class Shape:
    n_layers: int
    d_model: int
    n_q_heads: int
    n_kv_heads: int
    d_head: int
    d_ff: int
    rms_eps: float
    rope_theta: float
    dtype: str

    @property
    def d_q(self):
        return self.n_q_heads * self.d_head

    @property
    def d_kv(self):
        return self.n_kv_heads * self.d_head

    @property
    def params(self):
        return self.d_model * (2 * self.d_q + 2 * self.d_kv + 3 * self.d_ff)

    @property
    def elt(self):
        return 2 if self.dtype == "bf16" else 4

    @property
    def tdtype(self):
        return torch.bfloat16 if self.dtype == "bf16" else torch.float32


MODELS = {                                  # d_model, query heads, KV heads, head size, FFN, eps, storage
    "8b": (4096, 32, 8, 128, 14336, 1e-5, "bf16"),
    "70b": (8192, 64, 8, 128, 28672, 1e-5, "bf16"),
    "tiny": (256, 4, 4, 64, 688, 1e-6, "f32"),
}
VOCAB = 128256


def shape_of(case):
    d, q, kv, dh, ff, eps, dt = MODELS[case["model"]]
    return Shape(case["layers"], d, q, kv, dh, ff, eps, 500000.0, dt)


def listed():
    return [
        # the smallest stage: float32, 16 nodes behind a short context
        {"name": "tiny_f32", "kind": "tree", "model": "tiny", "layers": 2, "nodes": 16, "prefix": 128, "packed": False, "sizes": 1},
        # a stall: the true token enters as a level of its own
        {"name": "one_node_8b", "kind": "tree", "model": "8b", "layers": 1, "nodes": 1, "prefix": 512, "packed": True, "sizes": 1},
        # weights as they were loaded, without the re-layout; a ragged tree and context
        {"name": "tree37_rowmajor_8b", "kind": "tree", "model": "8b", "layers": 1, "nodes": 37, "prefix": 777, "packed": False,
         "sizes": 1},
        # the benchmark's step: 4 of 32 layers, a level's width of 64 nodes, context 2048 (a whole stage call)
        {"name": "tree64_8b", "kind": "tree", "model": "8b", "layers": 4, "nodes": 64, "prefix": 2048, "packed": True, "sizes": 1},
        # the 70B shape with a tree of two levels' width, context 4096
        {"name": "tree128_70b", "kind": "tree", "model": "70b", "layers": 2, "nodes": 128, "prefix": 4096, "packed": True,
         "sizes": 2},
        # a long context fed 1-8 nodes per step (a whole stage call)
        {"name": "stream_8b_32k", "kind": "stream", "model": "8b", "layers": 4, "prefix": 32768, "steps": 4, "max_new": 8,
         "packed": True, "sizes": 3},
        # 32 requests whose trees are all new: several hundred ragged rows
        {"name": "batch32_cold", "kind": "batch", "model": "8b", "layers": 2, "requests": 32, "t_lo": 8, "t_hi": 32,
         "p_lo": 512, "p_hi": 4096, "steady": False, "page": 0, "packed": True, "sizes": 4},
        # 32 requests in steady state, 1-8 nodes each, the cache in pages
        {"name": "batch32_steady_paged", "kind": "batch", "model": "8b", "layers": 2, "requests": 32, "t_lo": 1, "t_hi": 8,
         "p_lo": 512, "p_hi": 4096, "steady": True, "page": 64, "packed": True, "sizes": 4},
        # the last stage's output head over a level of 64 nodes
        {"name": "head_64", "kind": "head", "model": "8b", "layers": 1, "rows": 64, "packed": True},
        # stochastic decoding of a batch of 32 requests
        {"name": "sample_32", "kind": "verify", "model": "8b", "layers": 1, "requests": 32, "children": 8, "mode": "sample",
         "packed": True},
        # top-p verification of one request with a full level of root children
        {"name": "top_p_1", "kind": "verify", "model": "8b", "layers": 1, "requests": 1, "children": 64, "mode": "top_p",
         "packed": True},
        # the next level: 16 proposals for each of 64 bottom tokens, the best 64 kept and inserted
        {"name": "grow_64", "kind": "grow", "model": "8b", "layers": 1, "bottom": 64, "k": 16, "width": 64, "packed": True},
    ]


def _log_int(r, lo, hi):
    return int(round(math.exp(r.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    r = rng
    kind = r.choice(["tree", "tree", "tree", "stream", "batch", "batch", "head", "verify", "grow", "tiny"])
    if kind == "tiny":
        return {"kind": "tree", "model": "tiny", "layers": 2, "nodes": _log_int(r, 1, 64), "prefix": _log_int(r, 16, 512), "packed": False,
                "sizes": r.randrange(1 << 20)}
    if kind == "tree":
        model = r.choice(["8b", "8b", "70b"])
        return {"kind": "tree", "model": model, "layers": r.randint(1, 4 if model == "8b" else 2),
                "nodes": _log_int(r, 1, 256 if model == "8b" else 128), "prefix": _log_int(r, 64, 8192 if model == "8b" else 4096),
                "packed": r.random() < 0.75, "sizes": r.randrange(1 << 20)}
    if kind == "stream":
        return {"kind": "stream", "model": "8b", "layers": r.randint(1, 4), "prefix": _log_int(r, 2048, 32768), "steps": 4,
                "max_new": r.randint(1, 8), "packed": True, "sizes": r.randrange(1 << 20)}
    if kind == "batch":
        steady = r.random() < 0.5
        while True:
            case = {"kind": "batch", "model": "8b", "layers": r.randint(1, 2), "requests": _log_int(r, 2, 32),
                    "t_lo": 1 if steady else 8, "t_hi": 8 if steady else 32, "p_lo": 512, "p_hi": 4096, "steady": steady,
                    "page": r.choice([0, 64, 128]), "packed": r.random() < 0.75, "sizes": r.randrange(1 << 20)}
            if sum(_batch_sizes(case)[1]) <= sum(_batch_sizes(_LARGEST_BATCH)[1]):
                return case
    if kind == "head":
        return {"kind": "head", "model": "8b", "layers": 1, "rows": _log_int(r, 1, 64), "packed": r.random() < 0.75}
    if kind == "verify":
        mode = r.choice(["sample", "top_p", "relaxed"])
        return {"kind": "verify", "model": "8b", "layers": 1, "requests": _log_int(r, 1, 32), "children": _log_int(r, 4, 64),
                "mode": mode, "packed": True}
    bottom = _log_int(r, 1, 64)
    return {"kind": "grow", "model": "8b", "layers": 1, "bottom": bottom, "k": r.randint(1, 32), "width": _log_int(r, 8, 128), "packed": True}


_LARGEST_BATCH = {"requests": 32, "t_lo": 8, "t_hi": 32, "p_lo": 512, "p_hi": 4096, "sizes": 4}


# ---- inputs: values from the seed, sizes and the shapes of the trees from the case --------------------------------
def _gen(seed, what):
    return torch.Generator(device=DEV).manual_seed((int(seed) * 1000003 + what) % (1 << 62))


def _normal(g, sh, *size, std=1.0, mean=0.0):
    t = torch.randn(*size, generator=g, device=DEV, dtype=sh.tdtype)
    if std != 1.0:
        t *= std
    if mean:
        t += mean
    return t


def _layers(sh, seed):
    """Row-major weights of every layer: projections N(0, 0.02), norm gains 1 + N(0, 0.02)."""
    for l in range(sh.n_layers):
        g = _gen(seed, 100 + l)
        yield {"wqkv": _normal(g, sh, sh.d_q + 2 * sh.d_kv, sh.d_model, std=0.02),
               "wo": _normal(g, sh, sh.d_model, sh.d_q, std=0.02),
               "wgu": _normal(g, sh, 2 * sh.d_ff, sh.d_model, std=0.02),
               "wd": _normal(g, sh, sh.d_model, sh.d_ff, std=0.02),
               "norm1": _normal(g, sh, sh.d_model, std=0.02, mean=1.0),
               "norm2": _normal(g, sh, sh.d_model, std=0.02, mean=1.0)}


def _context(sh, seed, req, layer, P):
    """Rotated K and V of a request's committed context, [2, n_kv, P, d_head]."""
    return _normal(_gen(seed, 1000 + req * 64 + layer), sh, 2, sh.n_kv_heads, P, sh.d_head)


def _rows(sh, seed, what, n):
    return _normal(_gen(seed, 10 + what), sh, n, sh.d_model)


def _tree(r, n, max_children=4, max_levels=12, live=()):
    """n new nodes by sequential attachment under the root or any earlier node, with caps on children and levels."""
    parents, lev, kids = list(live), [], {-1: 0}
    for i, p in enumerate(parents):
        lev.append(0 if p < 0 else lev[p] + 1)
        kids[i] = 0
        kids[p] = kids.get(p, 0) + 1
    for _ in range(n):
        ok = [j for j in range(-1, len(parents)) if kids[j] < max_children and (j < 0 or lev[j] + 1 < max_levels)]
        p = r.choice(ok or [-1])
        kids[p] += 1
        kids[len(parents)] = 0
        lev.append(0 if p < 0 else lev[p] + 1)
        parents.append(p)
    return parents[len(live):]


def _one_tree(case):
    return _tree(random.Random("tree %d" % case["sizes"]), case["nodes"])


def _pruned(parents, node, accept):
    """(old indices of the tree nodes that stay, their new parents) after an accept of, or a drop at, `node`."""
    inside = []
    for i, p in enumerate(parents):
        inside.append(i == node or (p >= 0 and inside[p]))
    keep = [i for i in range(len(parents)) if (inside[i] and i != node if accept else not inside[i])]
    new = {o: k for k, o in enumerate(keep)}
    return keep, [new.get(parents[o], -1) for o in keep]


def _busiest_child(parents):
    """The root's child with the most nodes below it: the branch on which the tree has grown."""
    size = [1] * len(parents)
    for i in range(len(parents) - 1, -1, -1):
        if parents[i] >= 0:
            size[parents[i]] += size[i]
    return max((i for i, p in enumerate(parents) if p < 0), key=lambda i: size[i])


def _stream_plan(case):
    """Per step: parents of the new nodes, then (accept?, node)."""
    r = random.Random("stream %d" % case["sizes"])
    live, plan = [], []
    for _ in range(case["steps"]):
        new = [r.randint(-1, len(live) + k - 1) for k in range(r.randint(max(1, case["max_new"] // 2), case["max_new"]))]
        live = live + new
        accept = r.random() < 0.7
        node = _busiest_child(live) if accept else r.randrange(len(live))
        plan.append((new, accept, node))
        live = _pruned(live, node, accept)[1]
    return plan


def _batch_sizes(case):
    """(context lengths, new nodes, new nodes of the second level) of the requests."""
    r = random.Random("batch %d" % case["sizes"])
    R = range(case["requests"])
    return ([r.randint(case["p_lo"], case["p_hi"]) for _ in R], [r.randint(case["t_lo"], case["t_hi"]) for _ in R],
            [r.randint(case["t_lo"], case["t_hi"]) for _ in R])


def _batch_plan(case):
    """Per request: first tree, the node whose subtree is dropped, the nodes that follow."""
    r = random.Random("trees %d" % case["sizes"])
    out = []
    for n1, n2 in zip(*_batch_sizes(case)[1:]):
        first = _tree(r, n1, max_levels=6)
        node = r.randrange(n1)
        out.append((first, node, _tree(r, n2, max_levels=6, live=_pruned(first, node, False)[1])))
    return out


def _head(sh, seed):
    g = _gen(seed, 5)
    return {"norm": _normal(g, sh, sh.d_model, std=0.02, mean=1.0), "wvocab": _normal(g, sh, VOCAB, sh.d_model, std=0.02)}


def _head_rows(sh, seed, n, head):
    """Rows of the last layer that lean towards some two dozen tokens each, as a trained model's do: their logits stand
    a few units above the others.  Returns the rows and those tokens."""
    g = _gen(seed, 6)
    x = torch.randn(n, sh.d_model, generator=g, device=DEV)
    tok = torch.randint(0, VOCAB, (n, 24), generator=g, device=DEV)
    gain = 0.03 + 0.07 * torch.rand(n, 24, generator=g, device=DEV)
    for j in range(24):
        x += gain[:, j:j + 1] * head["wvocab"][tok[:, j]].float() / 0.02
    return x.to(sh.tdtype).contiguous(), tok


def _children(case, seed, tok):
    """Root children of every request (tokens, draft probabilities): half of them among the model's likely tokens."""
    r = random.Random("children %d" % seed)
    out = []
    for row in tok.tolist():
        t = [r.choice(row) if r.random() < 0.5 else r.randrange(VOCAB) for _ in range(case["children"])]
        out.append((t, [float(np.float32(r.uniform(0.01, 1.0))) for _ in t]))
    return out


def _uniforms(case, seed):
    r = random.Random("u %d" % seed)
    return [float(np.float32(r.random() * 0.999)) for _ in range(case["requests"])]


def _candidates(case, seed):
    g = _gen(seed, 7)
    tok = torch.randint(0, VOCAB, (case["bottom"], case["k"]), generator=g, device=DEV, dtype=torch.int32)
    prob = torch.rand(case["bottom"], case["k"], generator=g, device=DEV, dtype=torch.float32)
    prob = (prob ** 3).sort(dim=1, descending=True).values.contiguous()
    r = random.Random("grow %d" % seed)
    n = case["bottom"]
    return tok, prob, [r.randrange(VOCAB) for _ in range(n)], [float(np.float32(r.uniform(0.05, 1.0))) for _ in range(n)]


# ---- what the program holds before the call --------------------------------------------------------------------
_stream = None


def _own_stream():
    """A serving loop's stream: forward calls replay their graphs only on a stream that can be captured."""
    global _stream
    if _stream is None:
        torch.cuda.synchronize()
        _stream = torch.cuda.Stream(device=DEV)
    torch.cuda.set_stream(_stream)


def _stage(case, seed, slots, requests=1, rows=64, page=0):
    sh = shape_of(case)
    layers, flags = list(_layers(sh, seed)), 0
    if case["packed"]:
        layers, flags = [sp.pack_weights(sh, [w], DEV)[0] for w in layers], sp.SP_FLAG_PACKED_WEIGHTS
    if page:
        flags |= sp.SP_FLAG_PAGED_KV
    return sp.Stage(sh, layers, kv_slots=slots, max_requests=requests, max_batch_nodes=max(64, rows), flags=flags, page_slots=page)


def prepare(case, seed):
    _own_stream()
    sh, kind = shape_of(case), case["kind"]
    s = {"case": case, "sh": sh}
    if kind in ("tree", "stream"):
        P = case["prefix"]
        s["cap"] = P + 256 + 64
        s["stage"] = _stage(case, seed, s["cap"], rows=case.get("nodes", 8))
        kv = s["kv"] = s["stage"].kv_view()
        for l in range(sh.n_layers):
            kv[l, :, :, :P] = _context(sh, seed, 0, l, P)
        if kind == "tree":
            n = case["nodes"]
            r = random.Random("tokens %d" % seed)
            s["parents"] = _one_tree(case)
            s["tokens"], s["probs"] = [r.randrange(VOCAB) for _ in range(n)], [r.random() for _ in range(n)]
            s["accept"] = _busiest_child(s["parents"])
            s["x"] = _rows(sh, seed, 0, n)
            s["y"] = torch.empty_like(s["x"])
            s["nodes"] = list(range(n))
        else:
            s["plan"] = _stream_plan(case)
            s["x"] = [_rows(sh, seed, k, len(p[0])) for k, p in enumerate(s["plan"])]
            s["y"] = [torch.empty_like(x) for x in s["x"]]
        s["stage"].request_init(0, 0, s["cap"], P)
    elif kind == "batch":
        Ps, n1, n2 = _batch_sizes(case)
        s["plan"], s["ids"], pg = _batch_plan(case), list(range(case["requests"])), case["page"]
        room = [P + 64 for P in Ps]
        base, off = [], 0
        for c in room:
            base.append(0 if pg else off)
            off += -(-c // pg) * pg if pg else c
        R = len(Ps)
        st = s["stage"] = _stage(case, seed, off, requests=R + 2, rows=max(sum(n1), sum(n2)), page=pg)
        kv = st.kv_view()
        if pg:              # two requests that came and went: the pages are handed out of order from here on
            third = max(1, off // pg // 3) * pg
            for q in (R, R + 1):
                st.request_init(q, 0, third, third)
            for q in (R, R + 1):
                st.request_release(q)
        for q in s["ids"]:
            st.request_init(q, base[q], room[q], Ps[q])
            at = st.logical_slots(q, 0, Ps[q]) if pg else None
            for l in range(sh.n_layers):
                c = _context(sh, seed, q, l, Ps[q])
                if pg:
                    kv[l].index_copy_(2, at, c)
                else:
                    kv[l, :, :, base[q]:base[q] + Ps[q]] = c
        # where the cache of a request's tree lies (contiguous storage): views of the slab
        live = [len(p[0]) if not case["steady"] else len(_pruned(p[0], p[1], False)[0]) + len(p[2]) for p in s["plan"]]
        s["kv"] = None if pg else [kv[:, :, :, base[q] + Ps[q]:base[q] + Ps[q] + live[q]] for q in s["ids"]]
        s["x"] = [_rows(sh, seed, 0, sum(n1))] + ([_rows(sh, seed, 1, sum(n2))] if case["steady"] else [])
        s["y"] = [torch.empty_like(x) for x in s["x"]]
    elif kind == "head":
        n = case["rows"]
        st = s["stage"] = _stage(case, seed, 512, rows=n)
        head = _head(sh, seed)
        s["rows"], _ = _head_rows(sh, seed, n, head)
        st.request_init(0, 0, 512, 64)
        st.tree_insert(0, _tree(random.Random("tree %d" % seed), n))
        st.stage_forward([0], [0], [n], _rows(sh, seed, 0, n))
        s["head"] = dict(head, wvocab=sp.pack_matrix(head["wvocab"])) if case["packed"] else head
    elif kind == "verify":
        n = case["requests"]
        st = s["stage"] = _stage(case, seed, 256 * n, requests=n)
        head = _head(sh, seed)
        s["rows"], tok = _head_rows(sh, seed, n, head)
        s["ids"], s["u"] = list(range(n)), _uniforms(case, seed)
        for q, (t, p) in enumerate(_children(case, seed, tok)):
            st.request_init(q, 256 * q, 256, 64)
            st.tree_insert(q, [-1] * len(t), t, p)
        s["head"] = dict(head, wvocab=sp.pack_matrix(head["wvocab"])) if case["packed"] else head
    else:
        s["stage"] = _stage(case, seed, 512)
        s["cand"] = _candidates(case, seed)
        s["stage"].request_init(0, 0, 512, 64)
    torch.cuda.synchronize()
    return s


# ---- one pass ----------------------------------------------------------------------------------------------------
def run(s):
    case, st, kind = s["case"], s["stage"], s["case"]["kind"]
    if kind == "tree":
        n, P = case["nodes"], case["prefix"]
        st.request_init(0, 0, s["cap"], P)
        st.tree_insert(0, s["parents"], s["tokens"], s["probs"])
        st.stage_forward([0], [0], [n], s["x"], s["y"])
        live, commit = st.tree_prune(0, sp.SP_ACCEPT, s["accept"])
        rows, nodes = st.kv_compact(0, s["y"], s["nodes"])
        return {"y": s["y"][:rows], "nodes": np.asarray(nodes), "kv": s["kv"][:, :, :, P:P + commit + live]}
    if kind == "stream":
        P, out = case["prefix"], []
        st.request_init(0, 0, s["cap"], P)
        for (parents, accept, node), x, y in zip(s["plan"], s["x"], s["y"]):
            n = len(parents)
            first = st.tree_insert(0, parents)
            st.stage_forward([0], [first], [n], x, y)
            live, _ = st.tree_prune(0, sp.SP_ACCEPT if accept else sp.SP_DROP, node)
            rows, _ = st.kv_compact(0, y, list(range(first, first + n)))
            out.append(y[:rows])
        end = st.request_info(0)[0] + live
        return {"y": out, "kv": s["kv"][:, :, :, P:end]}
    if kind == "batch":
        ids, plan = s["ids"], s["plan"]
        st.tree_prune_batch(ids, [sp.SP_CLEAR] * len(ids), [0] * len(ids))
        st.kv_compact_batch(ids)
        first = st.tree_insert_batch(ids, [p[0] for p in plan])
        st.stage_forward(ids, first, [len(p[0]) for p in plan], s["x"][0], s["y"][0])
        if case["steady"]:
            st.tree_prune_batch(ids, [sp.SP_DROP] * len(ids), [p[1] for p in plan])
            st.kv_compact_batch(ids)
            first = st.tree_insert_batch(ids, [p[2] for p in plan])
            st.stage_forward(ids, first, [len(p[2]) for p in plan], s["x"][1], s["y"][1])
        return {"y": s["y"], "kv": s["kv"]}
    if kind == "head":
        pred, top = st.verify_head(s["head"], [0], [0], [case["rows"]], s["rows"], want_max=True)
        return {"pred": pred, "max": top}
    if kind == "verify":
        if case["mode"] == "sample":
            got = st.verify_sample(s["head"], s["ids"], s["rows"], 0.6, 0.9, 80, s["u"])
        else:
            got = st.verify_lossy(s["head"], s["ids"], s["rows"],
                                  sp.SP_VERIFY_TOP_P if case["mode"] == "top_p" else sp.SP_VERIFY_RELAXED, 0.9)
        return np.asarray(got)
    tok, prob, level_tok, level_prob = s["cand"]
    n = case["bottom"]
    st.tree_prune(0, sp.SP_CLEAR, 0)
    st.kv_compact(0)
    st.tree_insert(0, [-1] * n, level_tok, level_prob)
    parents, tokens, probs = st.tree_expand(0, list(range(n)), tok, prob, case["width"])
    first = st.tree_insert(0, parents, tokens, probs)
    return {"parents": np.asarray(parents), "tokens": np.asarray(tokens), "probs": np.asarray(probs, np.float32), "first": first}


# ---- what a pass cannot do without -------------------------------------------------------------------------------
def _forward_work(sh, M, spans, new):
    """One forward of M rows: weights, cache of the requests (spans: slots each sees), rows in and out, new cache rows."""
    kv = 2 * sh.d_kv * sh.elt
    nbytes = sh.n_layers * (sh.params * sh.elt + sum(spans) * kv) + 2 * M * sh.d_model * sh.elt
    flops = sh.n_layers * (2 * M * sh.params + 4 * sh.d_q * sum(n * s for n, s in zip(new, spans)))
    return nbytes, flops


def work(case):
    sh, kind = shape_of(case), case["kind"]
    if kind == "tree":
        b, f = _forward_work(sh, case["nodes"], [case["prefix"] + case["nodes"]], [case["nodes"]])
    elif kind == "stream":
        b = f = 0
        for new, _, _ in _stream_plan(case):
            x = _forward_work(sh, len(new), [case["prefix"] + len(new)], [len(new)])
            b, f = b + x[0], f + x[1]
    elif kind == "batch":
        Ps, n1, n2 = _batch_sizes(case)
        b, f = _forward_work(sh, sum(n1), [P + n for P, n in zip(Ps, n1)], n1)
        if case["steady"]:
            x = _forward_work(sh, sum(n2), [P + n for P, n in zip(Ps, n2)], n2)
            b, f = b + x[0], f + x[1]
    elif kind in ("head", "verify"):
        M = case["rows"] if kind == "head" else case["requests"]
        b, f = VOCAB * sh.d_model * sh.elt + M * sh.d_model * sh.elt, 2 * M * VOCAB * sh.d_model
    else:
        b = case["bottom"] * (case["k"] * 8 + 44) + case["width"] * (12 + 44)
        b += (case["bottom"] + case["width"]) * sh.n_layers * 2 * sh.d_kv * sh.elt
        f = case["bottom"] * case["k"]
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times what the library is off the float64 pass: 5e-3 of the rows in bf16 (storage of every
    intermediate tensor in bf16), 1e-7 in float32, 2e-4 of the winning logits (their rows are stored in bf16)."""
    if case["kind"] == "grow":
        return "exact"
    if case["kind"] == "verify":
        return {"differ": 0.04}
    if case["kind"] == "head":
        return {"rel": 0.001, "max": 0.005, "differ": 0.04}
    if case["model"] == "tiny":
        return {"rel": 1e-6, "max": 2e-5}
    return {"rel": 0.02, "max": 0.12}


# ---- the same pass in float64 --------------------------------------------------------------------------------------
class _Ref:
    """Requests of one stage in float64: cache per layer [2, n_kv, slots, d_head], live tree as a parent list."""

    def __init__(self, case, seed, prefixes):
        self.sh, self.seed = shape_of(case), seed
        self.P, self.parents = list(prefixes), [[] for _ in prefixes]
        self.kv = [[_context(self.sh, seed, q, l, P).double() for l in range(self.sh.n_layers)] for q, P in enumerate(prefixes)]

    def insert(self, q, parents):
        self.parents[q] = self.parents[q] + list(parents)

    def forward(self, news, x):
        """news: per request the number of its last nodes that are computed; x: their rows, request by request."""
        sh, h = self.sh, x.double()
        dh, half, g = sh.d_head, sh.d_head // 2, sh.n_q_heads // sh.n_kv_heads
        freq = sh.rope_theta ** (-torch.arange(half, device=DEV, dtype=torch.float64) * 2 / dh)
        pos, masks = [], []
        for q, n in enumerate(news):
            par, P = self.parents[q], self.P[q]
            T = len(par)
            up = np.zeros((T, T), bool)
            for i, p in enumerate(par):
                if p >= 0:
                    up[i] = up[p]
                up[i, i] = True
            pos += [P + int(up[i].sum()) - 1 for i in range(T - n, T)]
            m = np.ones((n, P + T), bool)
            m[:, P:] = up[T - n:]
            masks.append(torch.from_numpy(m).to(DEV))
        ang = torch.tensor(pos, device=DEV, dtype=torch.float64)[:, None] * freq
        cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]

        def norm(v, gain):
            return v * torch.rsqrt(v.square().mean(-1, keepdim=True) + sh.rms_eps) * gain.double()

        def rot(v):
            a, b = v[..., :half], v[..., half:]
            return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

        for l, w in enumerate(_layers(sh, self.seed)):
            qkv = norm(h, w["norm1"]) @ w["wqkv"].double().T
            q_ = rot(qkv[:, :sh.d_q].reshape(-1, sh.n_q_heads, dh))
            k_ = rot(qkv[:, sh.d_q:sh.d_q + sh.d_kv].reshape(-1, sh.n_kv_heads, dh))
            v_ = qkv[:, sh.d_q + sh.d_kv:].reshape(-1, sh.n_kv_heads, dh)
            att, at = [], 0
            for q, n in enumerate(news):
                new = torch.stack([k_[at:at + n], v_[at:at + n]]).transpose(1, 2)
                kv = self.kv[q][l] = torch.cat([self.kv[q][l], new], 2)
                qq = q_[at:at + n].reshape(n, sh.n_kv_heads, g, dh).transpose(0, 1).reshape(sh.n_kv_heads, n * g, dh).contiguous()
                sc = torch.bmm(qq, kv[0].transpose(1, 2).contiguous()) / math.sqrt(dh)
                sc = sc.masked_fill(~masks[q].repeat_interleave(g, 0)[None], -math.inf)
                o = torch.bmm(torch.softmax(sc, -1), kv[1].contiguous())
                att.append(o.reshape(sh.n_kv_heads, n, g, dh).transpose(0, 1).reshape(n, sh.d_q))
                at += n
            h = h + torch.cat(att) @ w["wo"].double().T
            gu = norm(h, w["norm2"]) @ w["wgu"].double().T
            h = h + (torch.nn.functional.silu(gu[:, :sh.d_ff]) * gu[:, sh.d_ff:]) @ w["wd"].double().T
        return h

    def prune(self, q, node, accept):
        """Returns the old indices that stay, committed ones first."""
        keep, parents = _pruned(self.parents[q], node, accept)
        path = []
        if accept:
            j = node
            while j >= 0:
                path.insert(0, j)
                j = self.parents[q][j]
        P, old = self.P[q], path + keep
        rows = torch.tensor(list(range(P)) + [P + j for j in old], device=DEV)
        for l in range(self.sh.n_layers):
            self.kv[q][l] = self.kv[q][l][:, :, rows]
        self.P[q], self.parents[q] = P + len(path), parents
        return path, keep

    def cache(self, q, lo):
        return torch.stack([c[:, :, lo:] for c in self.kv[q]])


def exact(case, seed):
    sh, kind = shape_of(case), case["kind"]
    if kind == "tree":
        n, P = case["nodes"], case["prefix"]
        parents = _one_tree(case)
        ref = _Ref(case, seed, [P])
        ref.insert(0, parents)
        y = ref.forward([n], _rows(sh, seed, 0, n))
        node = _busiest_child(parents)
        _, keep = ref.prune(0, node, True)
        new = {o: k for k, o in enumerate(keep)}
        rows = sorted(keep + [node])
        return {"y": y[rows], "nodes": np.asarray([new.get(o, -1) for o in rows]), "kv": ref.cache(0, P)}
    if kind == "stream":
        ref, out = _Ref(case, seed, [case["prefix"]]), []
        for k, (parents, accept, node) in enumerate(_stream_plan(case)):
            ref.insert(0, parents)
            T, n = len(ref.parents[0]), len(parents)
            y = ref.forward([n], _rows(sh, seed, k, n))
            path, keep = ref.prune(0, node, accept)
            # of the rows in flight those stay whose node stays, or is the one that was accepted
            rows = sorted(i - (T - n) for i in keep + ([node] if accept else []) if i >= T - n)
            out.append(y[rows])
        return {"y": out, "kv": ref.cache(0, case["prefix"])}
    if kind == "batch":
        Ps, n1, n2 = _batch_sizes(case)
        ref, plan, out = _Ref(case, seed, Ps), _batch_plan(case), []
        for q, p in enumerate(plan):
            ref.insert(q, p[0])
        out.append(ref.forward(n1, _rows(sh, seed, 0, sum(n1))))
        if case["steady"]:
            for q, p in enumerate(plan):
                ref.prune(q, p[1], False)
                ref.insert(q, p[2])
            out.append(ref.forward(n2, _rows(sh, seed, 1, sum(n2))))
        return {"y": out, "kv": None if case["page"] else [ref.cache(q, Ps[q]) for q in range(len(Ps))]}
    if kind == "grow":
        tok, prob, _, level_prob = _candidates(case, seed)
        p = prob.cpu().numpy()
        cum = (np.float32(1) * np.asarray(level_prob, np.float32))[:, None] * p
        order = np.sort(np.argsort(-cum.reshape(-1), kind="stable")[:case["width"]])
        return {"parents": order // case["k"], "tokens": tok.cpu().numpy().reshape(-1)[order].astype(np.int64),
                "probs": p.reshape(-1)[order], "first": case["bottom"]}
    n = case["rows"] if kind == "head" else case["requests"]
    head = _head(sh, seed)
    rows, tok = _head_rows(sh, seed, n, head)
    x = rows.double()
    x = x * torch.rsqrt(x.square().mean(-1, keepdim=True) + sh.rms_eps) * head["norm"].double()
    logits = torch.cat([x @ w.double().T for w in head["wvocab"].split(16384)], 1)
    top = logits.argmax(1)
    if kind == "head":
        return {"pred": top.int(), "max": logits.max(1).values}
    got = []
    for q, (t, draft) in enumerate(_children(case, seed, tok)):
        p = torch.softmax(logits[q] / (0.6 if case["mode"] == "sample" else 1.0), 0)
        val, idx = torch.sort(p, descending=True, stable=True)
        val, idx = val.cpu().numpy(), idx.cpu().numpy()
        m = int(np.searchsorted(np.cumsum(val), np.float64(np.float32(0.9)))) + 1
        if case["mode"] == "sample":
            c = np.cumsum(val[:min(m, 80)])
            token = int(idx[min(int(np.searchsorted(c, _uniforms(case, seed)[q] * c[-1], side="right")), len(c) - 1)])
            got.append((t.index(token) if token in t else -1, token))
        elif case["mode"] == "top_p":
            ok = set(idx[:m].tolist())
            fit = [i for i, v in enumerate(t) if v in ok]
            got.append((max(fit, key=lambda i: (draft[i], -i)) if fit else -1, int(top[q])))
        else:
            pt = p[torch.tensor(t, device=DEV)].cpu().numpy()
            got.append((int(np.argmax(pt)), int(top[q])))
    return np.asarray(got)
