"""What this library is asked to do in earnest: cases to time, each one pass of a decode round's (or a request's) part.

A case names the model shape (the measurement configurations of the repository), the part of the path and its sizes:

  verify    tree-masked attention of every target layer over that layer's own K/V cache (once per decode round)
  draft     drafting of one tree: per level the Eq. 1 projections with the cache append, the cross-attention of the
            frontier and the expansion of its logits; the final ranking of the candidates (once per decode round)
  accept    greedy acceptance and the commit of the accepted rows in the caches of every layer (once per decode round)
  sample    acceptance at a sampling temperature (once per decode round)
  compress  scores of the visual tokens, selection, gather of the kept rows (once per request)
  entropy   attention entropy of a layer over a prompt (once per prompt and layer while layers are being chosen)

Calls are made one after the other on torch's current stream with preallocated outputs and workspaces, as a serving
loop makes them.  Sequences of a batch have different lengths when "ragged" is set, as they do in serving.
"""
import math
import random

import numpy as np
import torch

import paper_2505_19201_amd as dream

# (query heads, KV heads, head_dim, hidden, layers, vocabulary, visual tokens, prompt length, kept fraction 1/n)
SHAPES = {
    "tiny": (4, 4, 64, 256, 1, 1000, 64, 96, 2),
    "llava": (32, 32, 128, 4096, 32, 32000, 576, 704, 4),
    "pixtral": (32, 8, 128, 5120, 40, 131072, 1024, 1280, 4),
    "gemma3": (16, 8, 256, 3840, 48, 262144, 256, 1280, 2),
    "smolvlm": (32, 32, 64, 2048, 24, 49152, 1088, 1600, 4),
}
DEPTH = 6            # depth of a drafted tree
MAX_VERIFY_BYTES = 11.0e9     # what the largest listed case moves
MAX_LOGIT_BYTES = 2.1e9
MAX_SCORE_PAIRS = 32 * 32 * 1600 * 1600


def listed():
    return [
        # the smallest call: the float32 configuration, one layer of a tree of 8 nodes
        dict(name="verify_tiny_f32", op="verify", shape="tiny", batch=1, prefix=96, tree=8, ragged=False, lse=True),
        # one sequence, all 32 layers, the 60-node tree: the ordinary decode round of a multi-head model
        dict(name="verify_llava_b1", op="verify", shape="llava", batch=1, prefix=704, tree=60, ragged=False, lse=False),
        # grouped queries, head_dim 256, four sequences of different odd lengths, the paper's tree of 32 drafted tokens
        dict(name="verify_gemma3_b4_t33", op="verify", shape="gemma3", batch=4, prefix=1283, tree=33, ragged=True, lse=False),
        # grouped queries by four, a small serving batch of long prompts
        dict(name="verify_pixtral_b8", op="verify", shape="pixtral", batch=8, prefix=1280, tree=60, ragged=True, lse=False),
        # the largest: a serving batch of 32 sequences
        dict(name="verify_smolvlm_b32", op="verify", shape="smolvlm", batch=32, prefix=1600, tree=60, ragged=False, lse=False),
        # drafting for one sequence (launches count) and for a batch of 8
        dict(name="draft_llava_b1", op="draft", shape="llava", batch=1, prefix=704, width=10, budget=59),
        dict(name="draft_smolvlm_b8", op="draft", shape="smolvlm", batch=8, prefix=1601, width=10, budget=59),
        # end of a round: a large vocabulary for one sequence
        dict(name="accept_gemma3_b1", op="accept", shape="gemma3", batch=1, prefix=1280, tree=60, logits="bf16"),
        # temperature 1 over float32 logits (what samplers are usually given), a few sequences
        dict(name="sample_pixtral_b4_f32", op="sample", shape="pixtral", batch=4, tree=60, logits="f32", temperature=1.0),
        # compression of one prompt, both passes; and of a batch whose prefill left the rows' log-sum-exps
        dict(name="compress_llava_b1", op="compress", shape="llava", batch=1, prefix=704, row_lse=False),
        dict(name="compress_smolvlm_b16_lse", op="compress", shape="smolvlm", batch=16, prefix=1600, row_lse=True),
        # attention entropy of one layer over one prompt of odd length
        dict(name="entropy_pixtral_b1", op="entropy", shape="pixtral", batch=1, prefix=1279),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(("verify", "verify", "verify", "draft", "accept", "sample", "compress", "entropy"))
    shape = rng.choice(("llava", "pixtral", "gemma3", "smolvlm"))
    batch = _log(rng, 1, 32)
    prefix = _log(rng, 200, 2400)
    if op == "verify":
        if rng.random() < 0.1:
            return dict(op=op, shape="tiny", batch=rng.randint(1, 2), prefix=rng.randint(40, 400), tree=rng.randint(4, 16),
                        ragged=False, lse=True)
        case = dict(op=op, shape=shape, batch=batch, prefix=prefix, tree=rng.randint(8, 64), ragged=rng.random() < 0.5,
                    lse=rng.random() < 0.2)
        while case["batch"] > 1 and work(case)["bytes"] > MAX_VERIFY_BYTES:
            case["batch"] -= 1
        return case
    if op == "draft":
        width = rng.randint(4, 10)
        return dict(op=op, shape=shape, batch=min(batch, 8), prefix=prefix, width=width, budget=rng.randint(24, 63))
    if op in ("accept", "sample"):
        case = dict(op=op, shape=shape, batch=batch, tree=rng.randint(8, 64), logits=rng.choice(("bf16", "f32")))
        if op == "accept":
            case["prefix"] = min(prefix, 1600)
            case["batch"] = min(batch, 16)
        else:
            case["temperature"] = rng.choice((0.7, 1.0))
        while case["batch"] > 1 and _logit_bytes(case) > MAX_LOGIT_BYTES:
            case["batch"] -= 1
        return case
    case = dict(op=op, shape=shape, batch=batch, prefix=max(prefix, 320))
    if op == "compress":
        case["row_lse"] = rng.random() < 0.5
    while case["batch"] > 1 and case["batch"] * SHAPES[shape][0] * case["prefix"] ** 2 > MAX_SCORE_PAIRS:
        case["batch"] -= 1
    return case


# ---- sizes -----------------------------------------------------------------------------------------------------------
def _logit_bytes(case):
    return case["batch"] * case["tree"] * SHAPES[case["shape"]][5] * (4 if case["logits"] == "f32" else 2)


def _lengths(case):
    """Prefix length of every sequence: the asked one, or spread over its upper half."""
    r = random.Random("lengths %d %d" % (case["batch"], case["prefix"]))
    return [case["prefix"] if not case.get("ragged") or b == 0 else r.randint(case["prefix"] // 2, case["prefix"])
            for b in range(case["batch"])]


def _visual(case):
    """Visual tokens of the prompt: the configuration's share of it."""
    s = SHAPES[case["shape"]]
    return case["prefix"] * s[6] // s[7]


def _levels(case):
    """Frontier size of every drafted level, candidates in the pool, and frontier nodes over all levels."""
    w = case["width"]
    sizes = [1] + [w] * (DEPTH - 1)
    return sizes, 1 + w * sum(sizes), sum(sizes)


# ---- inputs ----------------------------------------------------------------------------------------------------------
def _tree(r, n, depth=DEPTH):
    """Parents of a level-ordered draft tree of n nodes: levels of about equal size, better ranked parents get more children."""
    depth = min(depth, n - 1)
    sizes = [1] + [(n - 1) // depth + (l < (n - 1) % depth) for l in range(depth)]
    parent, start = [-1], 0
    for l in range(1, len(sizes)):
        weights = [1.0 / (i + 1) for i in range(sizes[l - 1])]
        picks = sorted(r.choices(range(sizes[l - 1]), weights, k=sizes[l]))
        picks[0] = 0
        parent += [start + p for p in picks]
        start += sizes[l - 1]
    return parent


def _tokens(r, parent, vocab):
    """Drafted tokens, distinct among siblings."""
    token, used = [], {}
    for p in parent:
        t = r.randrange(vocab)
        while t in used.setdefault(p, set()):
            t = r.randrange(vocab)
        used[p].add(t)
        token.append(t)
    return token


def _path(r, parent, depth):
    """A root-to-node path of the asked depth, or the deepest below it."""
    best = [0]
    for i in range(len(parent)):
        p, a = [], i
        while a >= 0:
            p.append(a)
            a = parent[a]
        if len(p) - 1 <= depth and (len(p) > len(best) or (len(p) == len(best) and r.random() < 0.3)):
            best = p[::-1]
    return best


class _Rand:
    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def normal(self, *shape, dtype=torch.bfloat16, scale=1.0):
        x = torch.empty(*shape, dtype=dtype, device="cuda").normal_(generator=self.gen)
        return x if scale == 1.0 else x.mul_(scale)

    def uniform(self, *shape):
        return torch.rand(*shape, generator=self.gen, device="cuda")


def _ints(v):
    return torch.tensor(np.asarray(v, dtype=np.int32), device="cuda")


def _cache_rows(n):
    """Row capacity of a cache that holds n live rows (whole pages of 64 rows)."""
    return (n + 63) // 64 * 64


def _dt(name):
    return (dream.F32, torch.float32) if name == "f32" else (dream.BF16, torch.bfloat16)


def _prepare_verify(case, rnd, r):
    hq, hkv, d, _, layers = SHAPES[case["shape"]][:5]
    b, t = case["batch"], case["tree"]
    code, tdt = _dt("f32" if case["shape"] == "tiny" else "bf16")
    lengths = _lengths(case)
    rows = _cache_rows(max(lengths) + t)
    s = dict(desc=dream.attn_desc(b, hq, hkv, d, code, rows), layers=layers, tree=t, max_kv=max(lengths) + t,
             prefix_len=_ints(lengths), parent=_ints([_tree(r, t) for _ in range(b)]),
             q=rnd.normal(layers, b, t, hq, d, dtype=tdt), k=rnd.normal(layers, b, hkv, rows, d, dtype=tdt),
             v=rnd.normal(layers, b, hkv, rows, d, dtype=tdt), out=torch.empty(layers, b, t, hq, d, dtype=tdt, device="cuda"),
             lse=torch.empty(layers, b, hq, t, device="cuda") if case["lse"] else None)
    s["ws"] = dream.alloc_workspace(dream.dream_tree_verify_attn_workspace(s["desc"], t, s["max_kv"]))
    s["calls"] = [(s["q"][l], s["k"][l], s["v"][l], s["out"][l], s["lse"][l] if case["lse"] else None) for l in range(layers)]
    return s


def _run_verify(s):
    for q, k, v, out, lse in s["calls"]:
        dream.dream_tree_verify_attn(s["desc"], q, k, v, s["prefix_len"], s["tree"], s["parent"], None, s["max_kv"], out, lse, s["ws"])
    return [s["out"], s["lse"]]


def _prepare_draft(case, rnd, r):
    hq, hkv, d, hidden, _, vocab = SHAPES[case["shape"]][:6]
    b, w, p = case["batch"], case["width"], case["prefix"]
    sizes, n_pool, n_nodes = _levels(case)
    rows = _cache_rows(p + n_nodes)
    desc = dream.attn_desc(b, hq, hkv, d, dream.BF16, rows)
    # the frontier nodes in level order: a level's nodes hang off nodes of the level before
    parents, pool_parents = [], []
    for _ in range(b):
        parent, start = [-1], 0
        for l in range(1, len(sizes)):
            parent += sorted(start + min(int(r.expovariate(0.5)), sizes[l - 1] - 1) for _ in range(sizes[l]))
            start += sizes[l - 1]
        parents.append(parent)
        # candidate pool: every frontier node proposes w tokens; a frontier node is itself one of the candidates proposed before
        pool, of_node, at = [-1], {0: 0}, 1
        for l in range(len(sizes)):
            first = sum(sizes[:l])
            kids = []
            for f in range(sizes[l]):
                kids += [at + f * w + j for j in range(w)]
                pool += [of_node[first + f]] * w
            at += sizes[l] * w
            for i, c in enumerate(sorted(r.sample(kids, w))):
                of_node[first + sizes[l] + i] = c
        pool_parents.append(pool)
    pool_parent = _ints(pool_parents)
    step = -rnd.uniform(b, n_pool) * 3.0 - 0.05          # log-probabilities: scores fall along every path
    score, anc = step.clone(), pool_parent.long()
    for _ in range(DEPTH):
        score += torch.where(anc > 0, step.gather(1, anc.clamp(min=0)), torch.zeros_like(step))
        anc = torch.where(anc > 0, pool_parent.long().gather(1, anc.clamp(min=0)), anc)
    s = dict(desc=desc, batch=b, hidden=hidden, heads=(hq, hkv), vocab=vocab, width=w, n_nodes=n_nodes, n_pool=n_pool, budget=case["budget"],
             max_kv=p + n_nodes, prefix_len=_ints([p] * b), parent=_ints(parents), pool_parent=pool_parent, pool_score=score,
             pool_token=_ints([[r.randrange(vocab) for _ in range(n_pool)] for _ in range(b)]),
             wq=rnd.normal(hq * d, hidden, scale=hidden ** -0.5), wk=rnd.normal(hkv * d, hidden, scale=hidden ** -0.5),
             wv=rnd.normal(hkv * d, hidden, scale=hidden ** -0.5), k=rnd.normal(b, hkv, rows, d), v=rnd.normal(b, hkv, rows, d), levels=[])
    cuda = dict(device="cuda")
    for l, f in enumerate(sizes):
        first = sum(sizes[:l])
        s["levels"].append(dict(
            f=f, node=_ints([list(range(first, first + f))] * b), e=rnd.normal(b, f, hidden), x=rnd.normal(b, f, hidden),
            logits=rnd.normal(b, f, vocab, scale=3.0), cum=(-(rnd.uniform(b, f) * 3.0 * (l + 1)).sort(dim=1)[0] if l else torch.zeros(b, f, **cuda)).contiguous(),
            q=torch.empty(b, f, hq, d, dtype=torch.bfloat16, **cuda), out=torch.empty(b, f, hq, d, dtype=torch.bfloat16, **cuda),
            token=torch.empty(b, f, w, dtype=torch.int32, **cuda), score=torch.empty(b, f, w, **cuda),
            frontier=torch.empty(b, w, dtype=torch.int32, **cuda)))
    n_tree = 1 + min(case["budget"], n_pool - 1)
    s["tree"] = [torch.empty(b, n_tree, dtype=torch.int32, **cuda) for _ in range(3)]
    s["ws_attn"] = dream.alloc_workspace(max(dream.dream_draft_xattn_workspace(desc, f, s["max_kv"]) for f in sizes))
    s["ws_tree"] = dream.alloc_workspace(max(dream.dream_tree_expand_workspace(b, f, vocab, w) for f in sizes))
    return s


def _run_draft(s):
    desc, b, (hq, hkv) = s["desc"], s["batch"], s["heads"]
    for lv in s["levels"]:
        dream.dream_project_rows_multi(desc, [(lv["e"], s["wq"], hq, None, None, lv["q"]),
                                              (lv["x"], s["wk"], hkv, s["prefix_len"], lv["node"], s["k"]),
                                              (lv["x"], s["wv"], hkv, s["prefix_len"], lv["node"], s["v"])], lv["f"], s["hidden"])
        dream.dream_draft_xattn(desc, lv["q"], s["k"], s["v"], s["prefix_len"], s["n_nodes"], s["parent"], lv["f"], lv["node"], s["max_kv"],
                                lv["out"], s["ws_attn"])
        dream.dream_tree_expand_level(lv["logits"], dream.BF16, b, lv["f"], s["vocab"], lv["cum"], s["width"], lv["token"], lv["score"],
                                      lv["frontier"], s["ws_tree"])
    n = dream.dream_tree_finalize(s["pool_score"], s["pool_parent"], s["pool_token"], b, s["n_pool"], s["budget"], *s["tree"])
    return [[lv[k] for lv in s["levels"] for k in ("q", "out", "token", "score", "frontier")], s["k"], s["v"], s["tree"], n]


def _prepare_accept(case, rnd, r):
    _, hkv, d, _, layers, vocab = SHAPES[case["shape"]][:6]
    b, t, p = case["batch"], case["tree"], case["prefix"]
    code, tdt = _dt(case["logits"])
    parents = [_tree(r, t) for _ in range(b)]
    tokens = [_tokens(r, parents[i], vocab) for i in range(b)]
    logits = rnd.normal(b, t, vocab, dtype=tdt)
    at = []      # the target follows a path of some depth: its greedy choice there is the next node's token
    for i in range(b):
        path = _path(r, parents[i], r.randint(0, DEPTH))
        at += [(i, x, tokens[i][y]) for x, y in zip(path, path[1:])]
    if at:
        i, x, y = (torch.tensor(v, device="cuda") for v in zip(*at))
        logits[i, x, y] += 16.0
    rows = _cache_rows(p + t)
    i32 = dict(dtype=torch.int32, device="cuda")
    s = dict(desc=dream.attn_desc(b, hkv, hkv, d, dream.BF16, rows), code=code, batch=b, t=t, vocab=vocab, logits=logits, token=_ints(tokens),
             parent=_ints(parents), prefix_len=_ints([p] * b), caches=rnd.normal(2 * layers, b, hkv, rows, d), argmax=torch.empty(b, t, **i32),
             length=torch.empty(b, **i32), path=torch.empty(b, DEPTH + 1, **i32), bonus=torch.empty(b, **i32), new_len=torch.empty(b, **i32),
             ws=dream.alloc_workspace(dream.dream_accept_path_workspace(b, t, vocab)))
    s["each"] = list(s["caches"])
    return s


def _run_accept(s):
    dream.dream_accept_path(s["logits"], s["code"], s["batch"], s["t"], s["vocab"], s["token"], s["parent"], DEPTH, s["argmax"], s["length"],
                            s["path"], s["bonus"], s["ws"])
    dream.dream_kv_commit(s["desc"], s["each"], s["prefix_len"], s["t"], s["path"], s["length"], s["new_len"])
    return [s["argmax"], s["length"], s["path"], s["bonus"], s["new_len"], s["caches"]]


def _prepare_sample(case, rnd, r):
    vocab = SHAPES[case["shape"]][5]
    b, t = case["batch"], case["tree"]
    code, tdt = _dt(case["logits"])
    parents = [_tree(r, t) for _ in range(b)]
    # peaked distributions, the draft close to the target; children are likely tokens of their parent's draft row
    target = rnd.normal(b, t, vocab, dtype=torch.float32, scale=3.0)
    draft = target + rnd.normal(b, t, vocab, dtype=torch.float32, scale=0.7)
    likely = draft.topk(t, dim=2)[1].cpu().numpy()
    tokens = []
    for i in range(b):
        seen, row = {}, []
        for p in parents[i]:
            n = seen[p] = seen.get(p, -1) + 1
            row.append(int(likely[i, max(p, 0), n]))
        tokens.append(row)
    i32 = dict(dtype=torch.int32, device="cuda")
    return dict(target=target.to(tdt), draft=draft.to(tdt), code=code, batch=b, t=t, vocab=vocab, token=_ints(tokens), parent=_ints(parents),
                u=rnd.uniform(b, t), u_bonus=rnd.uniform(b), temperature=case["temperature"], length=torch.empty(b, **i32),
                path=torch.empty(b, DEPTH + 1, **i32), bonus=torch.empty(b, **i32),
                ws=dream.alloc_workspace(dream.dream_spec_accept_workspace(b, t, vocab)))


def _run_sample(s):
    dream.dream_spec_accept(s["target"], s["draft"], s["code"], s["batch"], s["t"], s["vocab"], s["token"], s["parent"], s["u"], s["u_bonus"],
                            DEPTH, s["temperature"], s["length"], s["path"], s["bonus"], s["ws"])
    return [s["length"], s["path"], s["bonus"]]


def _prompt(case, rnd):
    """Queries and keys of a layer over the prompt: keys differ in how much attention they draw, as visual tokens do."""
    hq, hkv, d = SHAPES[case["shape"]][:3]
    b, p = case["batch"], case["prefix"]
    rows = _cache_rows(p + 64)
    q, k = rnd.normal(b, p, hq, d), rnd.normal(b, hkv, rows, d)
    q[..., 0] += d ** 0.25
    k[..., 0] += (rnd.normal(b, 1, rows, dtype=torch.float32) * d ** 0.25).to(torch.bfloat16)
    return q, k, dream.attn_desc(b, hq, hkv, d, dream.BF16, rows)


def _prepare_compress(case, rnd, r):
    hq, hkv, d, hidden = SHAPES[case["shape"]][:4]
    b, p, v, den = case["batch"], case["prefix"], _visual(case), SHAPES[case["shape"]][8]
    q, k, desc = _prompt(case, rnd)
    kept = (v + den // 2) // den
    s = dict(q=q, k=k, desc=desc, p=p, v=v, den=den, hidden=hidden, rows=rnd.normal(b, p, hidden), lse=None,
             scores=torch.empty(b, v, device="cuda"), kept=torch.empty(b, kept, dtype=torch.int32, device="cuda"),
             dst=torch.empty(b, kept, hidden, dtype=torch.bfloat16, device="cuda"))
    if case["row_lse"]:
        s["lse"] = torch.empty(b, hq, p, device="cuda")
        causal = torch.full((p, p), float("-inf"), device="cuda").triu(1)
        for i in range(b):          # one sequence and a KV head's query heads at a time, in float32
            for h in range(hq):
                x = q[i, :, h].float() @ k[i, h * hkv // hq, :p].float().t().contiguous()
                s["lse"][i, h] = torch.logsumexp(x * d ** -0.5 + causal, dim=1)
    s["ws"] = dream.alloc_workspace(dream.dream_visual_compress_workspace(desc, p, v))
    return s


def _run_compress(s):
    n = dream.dream_visual_compress(s["desc"], s["q"], None, s["p"], s["k"], s["p"], 0, s["v"], 1, s["den"], None, s["scores"], s["kept"],
                                    s["rows"], s["p"], s["dst"], s["hidden"], s["ws"], row_lse_in=s["lse"])
    return [s["scores"], s["kept"], s["dst"], n]


def _prepare_entropy(case, rnd, r):
    q, k, desc = _prompt(case, rnd)
    b, p = case["batch"], case["prefix"]
    return dict(q=q, k=k, desc=desc, p=p, rows=torch.empty(b, desc.n_q_heads, p, device="cuda"), ae=torch.empty(b, device="cuda"),
                ws=dream.alloc_workspace(dream.dream_attention_entropy_workspace(desc, p)))


def _run_entropy(s):
    dream.dream_attention_entropy(s["desc"], s["q"], None, s["p"], s["k"], s["p"], s["rows"], s["ae"], s["ws"])
    return [s["rows"], s["ae"]]


_PREPARE = dict(verify=_prepare_verify, draft=_prepare_draft, accept=_prepare_accept, sample=_prepare_sample, compress=_prepare_compress,
                entropy=_prepare_entropy)
_RUN = dict(verify=_run_verify, draft=_run_draft, accept=_run_accept, sample=_run_sample, compress=_run_compress, entropy=_run_entropy)


def prepare(case, seed):
    dream.load()
    dream.dream_init()
    return case["op"], _PREPARE[case["op"]](case, _Rand(seed), random.Random(seed))


def run(state):
    op, s = state
    return _RUN[op](s)


# ---- what a pass cannot do without -----------------------------------------------------------------------------------
def work(case):
    hq, hkv, d, hidden, layers, vocab = SHAPES[case["shape"]][:6]
    b, op = case["batch"], case["op"]
    if op == "verify":
        e, t = (4 if case["shape"] == "tiny" else 2), case["tree"]
        keys = sum(_lengths(case)) + b * t
        return dict(bytes=layers * (2 * keys * hkv * d * e + 2 * b * t * hq * d * e + (b * hq * t * 4 if case["lse"] else 0)),
                    flops=layers * 4 * keys * t * hq * d)
    if op == "draft":
        # every level depends on the one before it, so each reads the weights and the cache again
        sizes, n_pool, n_nodes = _levels(case)
        keys = case["prefix"] + n_nodes
        per_level = (hq + 2 * hkv) * d * hidden * 2 + 2 * b * keys * hkv * d * 2
        rows = b * sum(sizes)
        return dict(bytes=len(sizes) * per_level + rows * (2 * hidden * 2 + (3 * hq + 2 * hkv) * d * 2 + vocab * 2) + b * n_pool * 12,
                    flops=2 * rows * (hq + 2 * hkv) * d * hidden + 4 * rows * keys * hq * d)
    if op == "accept":
        # half of the drafted depth is accepted on average; its rows are read and written in every cache
        return dict(bytes=_logit_bytes(case) + 2 * layers * b * hkv * (1 + DEPTH // 2) * d * 2 * 2, flops=b * case["tree"] * vocab)
    if op == "sample":
        # target rows of every node and draft rows of the nodes with children (about half of them)
        return dict(bytes=1.5 * _logit_bytes(case), flops=1.5 * 4 * b * case["tree"] * vocab)
    p = case["prefix"]
    size = b * p * hq * d * 2 + b * p * hkv * d * 2
    pairs = b * hq * p * p / 2
    if op == "compress":
        v, den = _visual(case), SHAPES[case["shape"]][8]
        visual_pairs = b * hq * (p * v - v * v / 2)
        return dict(bytes=size + b * (v * 4 + (v // den) * (2 * hidden * 2 + 4)) + (b * hq * p * 4 if case["row_lse"] else 0),
                    flops=2 * d * (visual_pairs if case["row_lse"] else pairs + visual_pairs))
    return dict(bytes=size + b * hq * p * 4, flops=2 * d * pairs)


def tolerance(case):
    op = case["op"]
    if op == "verify":
        # bf16 outputs of bf16 probabilities (float32: sums of some hundred terms)
        return {"rel": 1e-5, "max": 1e-4} if case["shape"] == "tiny" else {"rel": 1e-2, "max": 0.1}
    if op == "draft":
        # bf16 rows as above; tokens and trees compare float32 scores, which may tie within rounding
        return {"rel": 1e-2, "max": 0.1, "differ": 0.002}
    if op == "accept":
        return "exact"
    if op == "sample":
        return {"rel": 0.0, "differ": 0.01}      # float32 probabilities decide whole numbers
    # float32 sums of exponentials of float32 scores over exact bf16 products
    return {"rel": 5e-5, "max": 1e-3, "differ": 0.002}
