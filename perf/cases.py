"""The decode-attention work that users of this framework have it do, as a list of measurable cases.

A case is one call (or one model step) through ``PlannedAttention``: a plan and page pools that a serving
loop holds, new queries, and the attention output of every request.  The listed cases cover the forests
the framework is for (one request, short chats, document question answering, trees of three and more
levels, irregular forests, very long shared prefixes, unshared batches, verification of drafted tokens),
MHA / GQA / MQA, all three head dimensions, both data types, several page sizes and layouts, and the plan
options in use.  ``draw`` gives more of the same ranges.

Page pools are seeded permutations with spare pages, as a pool looks after some hours of serving.  K and V
are N(0, 1); queries are scaled so that the logits spread with a standard deviation of two.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2505_17694_amd import PlannedAttention

DEVICE = "cuda:0"
FP16, BF16 = 0, 1                       # the framework's dtype codes
DTYPES = {FP16: torch.float16, BF16: torch.bfloat16}
SPARE_PAGES = 64
QUERY_SCALE = 2.0

DEFAULT = dict(share=1, schedule=0, fused=0, extensions=0)
CHOOSE = dict(share=2, schedule=2, fused=2, extensions=3)      # the library chooses plan, schedule and launches
TUNED = dict(share=1, schedule=0, fused=0, extensions=3)       # the prefix-shared plan with both solver extensions


def _case(tree, hq, hkv, d, dtype, page, layout, options, name=None, layers=0, **sizes):
    c = dict(tree=tree, hq=hq, hkv=hkv, d=d, dtype=dtype, page=page, layout=layout, layers=layers, **options, **sizes)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # four short chats behind one system prompt, a small MHA model: the latency of a call counts
        _case("two_level", 8, 8, 128, FP16, 16, "htd", CHOOSE, "small_chat_mha",
              root=1024, leaves=4, leaf_min=64, leaf_max=64, shape=1),
        # a single user, one context of odd length, nothing shared
        _case("unshared", 32, 8, 128, BF16, 16, "thd", DEFAULT, "single_request",
              leaves=1, leaf_min=8191, leaf_max=8191, shape=2),
        # questions on one document: a whole decoding step of a 32-layer model, which carries the plan
        # over to the lengths grown by one token and then runs every layer with it
        _case("two_level", 32, 8, 128, BF16, 16, "htd", TUNED, "docqa_step_32_layers", layers=32,
              root=4096, leaves=64, leaf_min=255, leaf_max=255, shape=3),
        # system prompt, 16 documents, 16 questions each of ragged length
        _case("three_level", 32, 8, 128, BF16, 16, "htd", TUNED, "three_level_documents",
              root=2048, mids=16, mid=8192, leaves=16, leaf_min=32, leaf_max=512, shape=4),
        # an irregular forest of 512 requests (agents, retries, few-shot variants)
        _case("random", 32, 8, 128, BF16, 16, "htd", CHOOSE, "irregular_forest",
              leaves=512, levels=5, median=512, leaf_min=16, leaf_max=32768, shape=1003),
        # 64 requests on one very long context, groups of eight
        _case("two_level", 64, 8, 128, BF16, 16, "htd", TUNED, "long_shared_context",
              root=131072, leaves=64, leaf_min=1024, leaf_max=1024, shape=6),
        # the largest: the same beside 64 unshared long contexts
        _case("mixed", 64, 8, 128, BF16, 16, "htd", TUNED, "long_shared_and_unshared",
              root=131072, leaves=64, leaf_min=1024, leaf_max=1024, others=64, other=32768, shape=7),
        # verification of 64 drafted tokens on each of 16 sequences, with visibility masks
        _case("drafted", 32, 8, 128, BF16, 16, "htd", TUNED, "verify_drafted_tokens",
              root=2048, leaves=16, leaf_min=8192, leaf_max=8192, drafted=64, shape=8),
        # continuous batching without shared prefixes: short ragged contexts, groups of seven, larger pages
        _case("unshared", 28, 4, 128, FP16, 64, "thd", DEFAULT, "ragged_unshared_batch",
              leaves=256, leaf_min=100, leaf_max=4000, shape=9),
        # one few-shot prompt under a tree of samples, all query heads on one KV head
        _case("kary", 32, 1, 128, BF16, 32, "htd", TUNED, "sampling_tree_mqa",
              arity=2, levels=6, node=4096, shape=10),
        # heads of 64 channels: documents and questions
        _case("three_level", 64, 8, 64, BF16, 16, "htd", TUNED, "documents_64_channels",
              root=2048, mids=16, mid=8192, leaves=8, leaf_min=32, leaf_max=512, shape=11),
        # heads of 256 channels: documents and questions
        _case("three_level", 16, 8, 256, BF16, 16, "htd", TUNED, "documents_256_channels",
              root=2048, mids=16, mid=8192, leaves=16, leaf_min=32, leaf_max=512, shape=12),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, even over its logarithm, odd as often as not."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    hq, hkv, d, dtype = rng.choice([(8, 8, 128, FP16), (32, 8, 128, BF16), (32, 8, 128, FP16), (64, 8, 128, BF16),
                                    (28, 4, 128, BF16), (32, 1, 128, BF16), (64, 8, 64, BF16), (32, 8, 64, FP16),
                                    (16, 8, 256, BF16), (32, 8, 256, BF16)])
    page, layout = rng.choice([16, 16, 32, 64]), rng.choice(["htd", "htd", "thd"])
    options = rng.choice([DEFAULT, TUNED, TUNED, CHOOSE])
    kinds = ["two_level", "three_level", "random", "unshared", "kary", "mixed"]
    if hq // hkv <= 16:
        kinds.append("drafted")
    tree = rng.choice(kinds)
    shape = rng.randrange(1, 1 << 30)
    layers = rng.choice([0, 0, 0, 8]) if tree == "two_level" else 0
    lo = _spread(rng, 16, 512)
    leaf = dict(leaf_min=lo, leaf_max=_spread(rng, lo, 4 * lo))
    if tree == "two_level":
        sizes = dict(root=_spread(rng, 1000, 40000 if layers == 0 else 6000), leaves=_spread(rng, 2, 80), **leaf)
    elif tree == "three_level":
        sizes = dict(root=_spread(rng, 500, 4000), mids=_spread(rng, 2, 20), mid=_spread(rng, 700, 9000),
                     leaves=_spread(rng, 2, 18), **leaf)
    elif tree == "random":
        sizes = dict(leaves=_spread(rng, 30, 600), levels=rng.randrange(3, 7), median=_spread(rng, 100, 700),
                     leaf_min=16, leaf_max=16384)
    elif tree == "unshared":
        sizes = dict(leaves=_spread(rng, 1, 200), leaf_min=_spread(rng, 60, 300), leaf_max=_spread(rng, 1000, 8000))
    elif tree == "kary":
        sizes = dict(arity=rng.randrange(2, 5), levels=rng.randrange(2, 5), node=_spread(rng, 300, 9000))
    elif tree == "mixed":
        sizes = dict(root=_spread(rng, 4000, 60000), leaves=_spread(rng, 4, 64), others=_spread(rng, 4, 32),
                     other=_spread(rng, 1000, 9000), **leaf)
    else:
        sizes = dict(root=_spread(rng, 200, 3000), leaves=_spread(rng, 2, 18), leaf_min=_spread(rng, 500, 2000),
                     leaf_max=_spread(rng, 2000, 9000), drafted=rng.choice([3, 4, 8, 16, 31, 48, 64]))
    return _case(tree, hq, hkv, d, dtype, page, layout, options, layers=layers, shape=shape, **sizes)


# ---- forests: of the case alone, so that every seed asks for the same work -----------------------------


def _forest(c):
    """parent, node_len, req_node and, for drafted tokens, req_mask_off and req_mask."""
    rng = np.random.Generator(np.random.PCG64(c["shape"]))
    parent, length, last, masks = [], [], [], []

    def node(above, tokens):
        parent.append(above)
        length.append(int(tokens))
        return len(parent) - 1

    def leaf(above):
        last.append(node(above, rng.integers(c["leaf_min"], c["leaf_max"] + 1)))

    kind = c["tree"]
    if kind in ("two_level", "mixed"):
        root = node(-1, c["root"])
        for _ in range(c["leaves"]):
            leaf(root)
        for _ in range(c.get("others", 0)):
            last.append(node(-1, c["other"]))
    elif kind == "three_level":
        root = node(-1, c["root"])
        for _ in range(c["mids"]):
            mid = node(root, c["mid"])
            for _ in range(c["leaves"]):
                leaf(mid)
    elif kind == "unshared":
        for _ in range(c["leaves"]):
            leaf(-1)
    elif kind == "kary":
        level = [node(-1, c["node"])]
        for _ in range(c["levels"] - 1):
            level = [node(p, c["node"]) for p in level for _ in range(c["arity"])]
        last = level
    elif kind == "random":
        # breadth first; a node below the last level gets 1 + Poisson(2) children until there are enough leaves
        level_of, children, queue, at, leaves = [], [], [], 0, 0
        while leaves < c["leaves"]:
            if at == len(queue):
                queue.append(node(-1, 1))
                level_of.append(1)
                children.append(0)
                leaves += 1
                continue
            n = queue[at]
            at += 1
            if level_of[n] >= c["levels"]:
                continue
            children[n] = min(1 + int(rng.poisson(2.0)), c["leaves"] - leaves + 1)
            for _ in range(children[n]):
                queue.append(node(n, 1))
                level_of.append(level_of[n] + 1)
                children.append(0)
            leaves += children[n] - 1
        z = rng.standard_normal(len(parent))
        length = np.clip(np.rint(c["median"] * np.exp(z)), c["leaf_min"], c["leaf_max"]).astype(int).tolist()
        last = [n for n in range(len(parent)) if children[n] == 0]
    elif kind == "drafted":
        # per sequence one query for its newest token and one for each drafted token; a drafted token
        # follows the newest branch or an earlier token, and its query sees its own branch
        root, words = node(-1, c["root"]), (c["drafted"] + 31) // 32
        for _ in range(c["leaves"]):
            leaf(root)
            masks.append([])
            draft = node(last[-1], c["drafted"])
            after = []
            for k in range(c["drafted"]):
                after.append(k - 1 if rng.random() < 0.5 else int(rng.integers(-1, k)) if k else -1)
                bits, t = [0] * words, k
                while t >= 0:
                    bits[t // 32] |= 1 << (t % 32)
                    t = after[t]
                last.append(draft)
                masks.append(bits)
    else:
        raise ValueError(kind)
    f = SimpleNamespace(parent=np.array(parent, np.int32), node_len=np.array(length, np.int32),
                        req_node=np.array(last, np.int32), req_mask_off=None, req_mask=None)
    if masks:
        f.req_mask_off = np.concatenate([[0], np.cumsum([len(m) for m in masks])]).astype(np.int32)
        f.req_mask = np.array([w for m in masks for w in m], np.uint32)
    return f


def _grown(f):
    """The forest's lengths after one more decoding step: every request's last node holds one token more."""
    n = f.node_len.copy()
    n[np.unique(f.req_node)] += 1
    return n


def _requests_of_nodes(f):
    """Per node, the requests whose path holds it."""
    of = [[] for _ in f.parent]
    for r, n in enumerate(f.req_node):
        while n >= 0:
            of[n].append(r)
            n = f.parent[n]
    return of


# ---- what a program has in hand, the call, its cost ------------------------------------------------------


def _paged(c, node_len, seed):
    """Every node owns whole pages; physical pages in a seeded order.  A node has a page for its next token."""
    ps, h, d = c["page"], c["hkv"], c["d"]
    off = np.concatenate([[0], np.cumsum(node_len // ps + 1 if c["layers"] else (node_len + ps - 1) // ps)])
    total = int(off[-1]) + SPARE_PAGES
    ids = np.random.Generator(np.random.PCG64(seed)).permutation(total)[:int(off[-1])]
    token, head = (h * d, d) if c["layout"] == "thd" else (d, ps * d)
    return SimpleNamespace(node_page_off=off.astype(np.int32), page_ids=ids.astype(np.int32), num_pages=total,
                           page_stride=ps * h * d, token_stride=token, head_stride=head)


def _tensors(c, f, paged, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    ps, h, d = c["page"], c["hkv"], c["d"]
    shape = (paged.num_pages, ps, h, d) if c["layout"] == "thd" else (paged.num_pages, h, ps, d)
    layers = []
    for _ in range(max(1, c["layers"])):
        k = torch.empty(shape, dtype=DTYPES[c["dtype"]], device=DEVICE).normal_(generator=gen)
        v = torch.empty(shape, dtype=DTYPES[c["dtype"]], device=DEVICE).normal_(generator=gen)
        q = torch.empty((len(f.req_node), c["hq"], d), dtype=DTYPES[c["dtype"]], device=DEVICE)
        layers.append((q.normal_(0.0, QUERY_SCALE, generator=gen), k, v))
    return layers


def prepare(case, seed):
    f = _forest(case)
    paged = _paged(case, f.node_len, seed)
    head = SimpleNamespace(num_q_heads=case["hq"], num_kv_heads=case["hkv"], head_dim=case["d"], dtype=case["dtype"],
                           page_size=case["page"], scale=float(np.float32(1.0 / math.sqrt(case["d"]))))
    plan = PlannedAttention(f, paged, head, device=DEVICE, share=case["share"], schedule=case["schedule"],
                            fused=case["fused"], extensions=case["extensions"])
    return SimpleNamespace(plan=plan, layers=_tensors(case, f, paged, seed),
                           grown=_grown(f) if case["layers"] else None)


def run(state):
    if state.grown is None:
        q, k, v = state.layers[0]
        return state.plan.decode(q, k, v)
    state.plan.refresh(state.grown)
    return [state.plan.decode(q, k, v) for q, k, v in state.layers]


def work(case):
    f = _forest(case)
    lens = _grown(f) if case["layers"] else f.node_len
    requests = np.array([len(r) for r in _requests_of_nodes(f)], np.int64)
    layers = max(1, case["layers"])
    pairs = int((requests * lens).sum())                    # (request, token) pairs
    if f.req_mask is not None:                              # of a masked node a query sees its own branch only
        masked = np.flatnonzero(np.diff(f.req_mask_off))
        pairs -= int(f.node_len[f.req_node[masked]].sum())
        pairs += sum(bin(int(w)).count("1") for w in f.req_mask)
    kv = int(lens[requests > 0].sum()) * case["hkv"] * case["d"] * 4
    rows = len(f.req_node) * case["hq"] * case["d"] * 4     # queries in, outputs out
    return {"bytes": layers * (kv + rows), "flops": layers * 4 * pairs * case["hq"] * case["d"]}


def tolerance(case):
    # the probabilities and the output are rounded to 16 bits: 2.3e-3 (bf16) and 2.6e-4 (fp16) off the 64-bit
    # values as measured, stated about four times
    return {"rel": 1e-2} if case["dtype"] == BF16 else {"rel": 1.2e-3}


def exact(case, seed):
    f = _forest(case)
    paged = _paged(case, f.node_len, seed)
    lens = _grown(f) if case["layers"] else f.node_len
    outs = [_attention(case, f, paged, lens, *x) for x in _tensors(case, f, paged, seed)]
    return outs if case["layers"] else outs[0]


def _attention(c, f, paged, lens, q, k_pool, v_pool, chunk=8192):
    """softmax(scale q K^T) V in 64 bits, node by node, with the usual merge of partial softmaxes."""
    b, hq, d, h = len(f.req_node), c["hq"], c["d"], c["hkv"]
    g, ps = hq // h, c["page"]
    scale = float(np.float32(1.0 / math.sqrt(d)))
    q64 = q.double().view(b, h, g, d).permute(1, 0, 2, 3)                       # [h, b, g, d]
    top = torch.full((h, b, g), -math.inf, dtype=torch.float64, device=DEVICE)
    total = torch.zeros((h, b, g), dtype=torch.float64, device=DEVICE)
    out = torch.zeros((h, b, g, d), dtype=torch.float64, device=DEVICE)
    ids = torch.from_numpy(paged.page_ids.astype(np.int64)).to(DEVICE)

    def rows_of(pool, n, a, e):
        x = pool[ids[paged.node_page_off[n] + a // ps:paged.node_page_off[n] + (e + ps - 1) // ps]]
        x = x if c["layout"] == "thd" else x.transpose(1, 2)                    # [pages, ps, h, d]
        return x.reshape(-1, h, d)[:e - a].double().permute(1, 0, 2).contiguous()

    for n, requests in enumerate(_requests_of_nodes(f)):
        if not requests:
            continue
        r = torch.tensor(requests, device=DEVICE)
        seen = None
        if f.req_mask is not None and any(f.req_mask_off[x + 1] > f.req_mask_off[x] and f.req_node[x] == n for x in requests):
            bits = np.stack([f.req_mask[f.req_mask_off[x]:f.req_mask_off[x + 1]] for x in requests])
            t = np.arange(lens[n])
            seen = torch.from_numpy(((bits[:, t // 32] >> (t % 32).astype(np.uint32)) & 1).astype(bool)).to(DEVICE)
        for a in range(0, int(lens[n]), chunk):
            e = min(a + chunk, int(lens[n]))
            k, v = rows_of(k_pool, n, a, e), rows_of(v_pool, n, a, e)
            for part in torch.split(r, max(1, (1 << 26) // (g * h * (e - a)))):
                s = torch.matmul(q64[:, part].reshape(h, -1, d), k.transpose(1, 2).contiguous()) * scale
                s = s.view(h, len(part), g, e - a)
                if seen is not None:
                    s.masked_fill_(~seen[torch.isin(r, part)][None, :, None, a:e], -math.inf)
                m = torch.maximum(top[:, part], s.amax(-1))
                p = torch.exp(s - m[..., None])
                w = torch.exp(top[:, part] - m)
                total[:, part] = total[:, part] * w + p.sum(-1)
                o = torch.matmul(p.view(h, -1, e - a), v).view(h, len(part), g, d)
                out[:, part] = out[:, part] * w[..., None] + o
                top[:, part] = m
    return (out / total[..., None]).permute(1, 0, 2, 3).reshape(b, hq, d)
