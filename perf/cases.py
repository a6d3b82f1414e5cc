"""The work whose time is measured: decoding steps, prompt passes and the single stages around them, through the public
entry points of paper_2503_14153_amd.

A case is a dict of plain values. Its "kind" says which entry points a pass goes through:

  step     one decoding step of `batch` sequences whose caches hold `rows_lo` .. `rows_hi` committed rows (ragged):
           sd_spec_step with a candidate tree of `nodes` nodes, sd_greedy_step for nodes = 1. Returns the logits of
           every node, the draft heads' logits and the emitted tokens.
  prefill  prompts of `rows_lo` .. `rows_hi` tokens per sequence through the model into an empty cache; returns the
           last layer's key and value rows of every sequence.
  accept   sampling decoding's own stages on given logits: typical acceptance with the fragment cut, and the draw of
           one token per sequence.
  rows     a prefix of `rows_lo` rows restored into the cache of every sequence, layer by layer (saved rows of a shared
           prompt), then saved again.

Models have random weights of the shapes in workload/configs.py (the 7B-shaped and 13B-shaped decoders, the small
float32 one). One case runs the 7B shape at its full 32 layers; the others run a few layers of the same width, which is
the same kernels on the same operands per layer, and keeps the comparison of their outputs sharp.

A pass starts by putting the sequences back to where they were (length and carried draft), so that it can be repeated;
the candidates are random ids, so that which of them are accepted does not hang on ties between nearly equal logits.
"""
import math
from dataclasses import dataclass

import torch

import paper_2503_14153_amd as sd

DEV = "cuda"
STD = 0.02                     # weights ~ N(0, 0.02^2), gains 1


@dataclass(frozen=True)
class Shape:
    n_layers: int
    d_model: int
    n_heads: int
    head_dim: int
    d_ffn: int
    vocab: int
    n_medusa: int
    topk: int
    dtype: str
    rope_theta: float
    rms_eps: float = 1e-5


# width: (d_model, heads, head_dim, d_ffn, vocab, dtype, rope_theta, top-k), as workload/configs.py has them
WIDTHS = {
    "tiny": (256, 4, 64, 688, 1024, "f32", 1e4, 4),
    "7b": (4096, 32, 128, 11008, 32016, "bf16", 1e6, 10),
    "13b": (5120, 40, 128, 13824, 32016, "bf16", 1e6, 10),
}


def shape_of(c):
    d, nh, hd, F, V, dt, theta, k = WIDTHS[c["width"]]
    return Shape(c["layers"], d, nh, hd, F, V, c["heads"], k, dt, theta)


def step(name, width, layers, heads, batch, nodes, rows_lo, rows_hi):
    return {"name": name, "kind": "step", "width": width, "layers": layers, "heads": heads, "batch": batch, "nodes": nodes,
            "rows_lo": rows_lo, "rows_hi": rows_hi}


def listed():
    return [
        # the small float32 configuration: launches and latency, no bandwidth
        step("tiny-f32-tree16", "tiny", 2, 3, 1, 16, 64, 64),
        # the headline: one whole step of the 7B-shaped model, 64-node tree, a few hundred committed rows
        step("7b-full-tree64", "7b", 32, 4, 1, 64, 700, 700),
        # plain next-token decoding, one sequence: the baseline every speculative run is compared with
        step("7b-plain", "7b", 4, 4, 1, 1, 1000, 1000),
        # plain next-token decoding of a served batch
        step("7b-plain-batch8", "7b", 4, 4, 8, 1, 1024, 4096),
        # a served batch with small trees (acceptance per verified token is best there), odd in every size
        step("7b-batch5-tree12", "7b", 4, 3, 5, 12, 150, 2100),
        # the batched configuration: eight ragged sequences, 32-node trees
        step("7b-batch8-tree32", "7b", 4, 4, 8, 32, 1024, 4096),
        # the 13B-shaped configuration: 128-node tree over 4096 rows
        step("13b-tree128", "13b", 4, 5, 1, 128, 4096, 4096),
        # the paper's ten heads with the largest tree
        step("7b-heads10-tree256", "7b", 4, 10, 1, 256, 512, 512),
        # long context
        step("7b-long-tree64", "7b", 4, 4, 1, 64, 16384, 16384),
        # a prompt of ordinary length, not a multiple of anything
        {"name": "7b-prefill", "kind": "prefill", "width": "7b", "layers": 4, "heads": 4, "batch": 1, "rows_lo": 1500, "rows_hi": 1500},
        # what sampling decoding adds to a batched step
        {"name": "7b-accept-sample", "kind": "accept", "heads": 4, "batch": 8, "nodes": 32, "vocab": 32016},
        # a cached prefix of an odd length moved in and out of the cache
        {"name": "7b-rows", "kind": "rows", "width": "7b", "layers": 4, "heads": 4, "batch": 2, "rows_lo": 1003, "rows_hi": 1003},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["step", "prefill", "accept", "rows"], [8, 3, 1, 1])[0]
    if kind == "accept":
        return {"kind": kind, "heads": rng.randint(3, 10), "batch": rng.randint(1, 16), "nodes": rng.randint(2, 64),
                "vocab": _log(rng, 1000, 40000)}
    heads = rng.randint(3, 10)
    if kind == "rows":
        n = _log(rng, 20, 2000)
        return {"kind": kind, "width": "7b", "layers": rng.randint(1, 4), "heads": heads, "batch": rng.randint(1, 3),
                "rows_lo": n, "rows_hi": n}
    width = rng.choices(["7b", "13b", "tiny"], [6, 2, 2])[0]
    layers = rng.randint(2, 4)
    if kind == "prefill":
        batch = rng.randint(1, 4)
        lo = _log(rng, 20, 1500 // batch)
        return {"kind": kind, "width": width, "layers": 2 if width == "13b" else layers, "heads": heads, "batch": batch,
                "rows_lo": lo, "rows_hi": _log(rng, lo, 1500 // batch)}
    if rng.random() < 0.3:
        nodes = 1
    else:
        nodes = min(_log(rng, 4, 256), 60 if width == "tiny" else 256)       # (three heads, top-4: 85 nodes at most)
    batch = rng.randint(1, min(8, 256 // (-(-nodes // 32) * 32)))
    lo = _log(rng, 16, 200 if width == "tiny" else 4096)
    c = step("", width, layers, 3 if width == "tiny" else heads, batch, nodes, lo, _log(rng, lo, 400 if width == "tiny" else 6000))
    del c["name"]
    return c


# --------------------------------------------------------------------------------------------- inputs from the seed
def gen(seed, tag, device=DEV):
    """A generator of its own for every input: tag is a small whole number."""
    g = torch.Generator(device=device)
    g.manual_seed(seed * 100003 + tag)
    return g


def normal(seed, tag, shape, std, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=gen(seed, tag))


def dtype_of(s):
    return torch.bfloat16 if s.dtype == "bf16" else torch.float32


def weight(s, seed, name):
    """One weight tensor [out, in]; norms' gains are 1, the draft heads have a small bias."""
    d, F, V, dt = s.d_model, s.d_ffn, s.vocab, dtype_of(s)
    base = name.split(".")[-1]
    if base.endswith("norm"):
        return torch.ones(d, dtype=dt, device=DEV)
    order = ["wqkv", "wo", "w_gate", "w_up", "w_down"]
    if name in ("embed", "lm_head"):
        return normal(seed, 1 if name == "embed" else 2, (V, d), STD, dt)
    if name.startswith("medusa"):
        i = int(name[6:].split(".")[0])
        return normal(seed, 10 + 2 * i, (d, d), STD, dt) if base == "w" else normal(seed, 11 + 2 * i, (d,), 0.1, dt)
    layer = int(name[1:].split(".")[0])
    shapes = {"wqkv": (3 * d, d), "wo": (d, d), "w_gate": (F, d), "w_up": (F, d), "w_down": (d, F)}
    return normal(seed, 100 + 8 * layer + order.index(base), shapes[base], STD, dt)


def weight_names(s):
    names = ["embed", "lm_head", "final_norm"]
    for l in range(s.n_layers):
        names += ["l%d.%s" % (l, k) for k in ("attn_norm", "wqkv", "wo", "ffn_norm", "w_gate", "w_up", "w_down")]
    for i in range(s.n_medusa):
        names += ["medusa%d.w" % i, "medusa%d.b" % i]
    return names


def lengths(c):
    """Rows per sequence: ragged, the same for every seed (they are sizes)."""
    g = torch.Generator().manual_seed(c["rows_lo"] * 7919 + c["rows_hi"])
    n = torch.randint(c["rows_lo"], max(c["rows_hi"], c["rows_lo"]) + 1, (c["batch"],), generator=g)
    if c["batch"] > 1:
        n[0], n[-1] = c["rows_hi"], c["rows_lo"]           # both ends occur
    return [int(x) for x in n]


def cache_rows(s, seed, layer, b, n):
    """Already rotated keys and values that stand for a processed prompt: N(0, 0.5^2)."""
    k = normal(seed, 10000 + 64 * layer + 2 * b, (n, s.n_heads, s.head_dim), 0.5, dtype_of(s))
    v = normal(seed, 10001 + 64 * layer + 2 * b, (n, s.n_heads, s.head_dim), 0.5, dtype_of(s))
    return k, v


def tree_of(nodes, heads, topk):
    """Best-first candidate tree: a node reached through head ranks r_1 .. r_d scores sum(r) + 0.75 d; the `nodes` lowest
    scores are kept, depth by depth. (parent, depth, rank)."""
    level, every = [()], [()]
    for _ in range(heads):
        level = sorted((t + (r,) for t in level for r in range(topk)), key=lambda t: (sum(t), t))[:nodes]
        every += level
    every.sort(key=lambda t: (sum(t) + 0.75 * len(t), len(t), t))
    kept = sorted(every[:nodes], key=lambda t: (len(t), t))
    at = {t: i for i, t in enumerate(kept)}
    return [at[t[:-1]] if t else -1 for t in kept], [len(t) for t in kept], [t[-1] if t else 0 for t in kept]


def drafts(s, c, seed):
    g = gen(seed, 20000)
    root = torch.randint(0, s.vocab, (c["batch"],), generator=g, device=DEV, dtype=torch.int32)
    first = torch.randint(0, s.vocab, (c["batch"], s.n_medusa, 1), generator=g, device=DEV, dtype=torch.int32)
    cand = (first + 37 * torch.arange(s.topk, device=DEV, dtype=torch.int32)) % s.vocab       # distinct ids per head
    return root, cand.contiguous()


def stop_words(vocab, seed):
    """One id in five is syntactically significant."""
    bits = (torch.rand((vocab + 31) // 32, 32, generator=gen(seed, 20001), device=DEV) < 0.2).to(torch.int64)
    return (bits << torch.arange(32, device=DEV)).sum(1).to(torch.int32)


class State:
    pass


def prepare(case, seed):
    c, st = case, State()
    st.case = c
    if c["kind"] == "accept":
        return prepare_accept(c, seed, st)
    s = shape_of(c)
    weights = {n: weight(s, seed, n) for n in weight_names(s)}
    st.model = sd.Model(s, weights, max_rows=256)
    del weights
    st.lens = lengths(c)
    cap = max(st.lens) + s.n_medusa + 2
    st.kv = sd.KVCache(st.model, c["batch"], cap)
    if c["kind"] == "rows":
        st.rows = [[cache_rows(s, seed, l, b, st.lens[b]) for b in range(c["batch"])] for l in range(s.n_layers)]
    elif c["kind"] == "prefill":
        st.tokens = torch.randint(0, s.vocab, (sum(st.lens),), generator=gen(seed, 20002), device=DEV, dtype=torch.int32)
    else:
        for l in range(s.n_layers):
            for b, n in enumerate(st.lens):
                st.kv.write_rows(l, b, 0, *cache_rows(s, seed, l, b, n))
        torch.cuda.synchronize()
        st.kv.set_len(st.lens)
        st.root, st.cand = drafts(s, c, seed)
        st.stop = stop_words(s.vocab, seed)
        if c["nodes"] > 1:
            st.tree = sd.Tree(*tree_of(c["nodes"], s.n_medusa, s.topk), s.n_medusa, s.topk)
    return st


def run(st):
    c = st.case
    if c["kind"] == "step":
        st.kv.set_len(st.lens)
        st.kv.set_draft(st.root, st.cand)
        if c["nodes"] == 1:
            out = sd.greedy_step(st.model, st.kv, want_logits=True, want_head_logits=True)
        else:
            out = sd.spec_step(st.model, st.kv, st.tree, st.stop, want_logits=True, want_head_logits=True)
        return {"logits": out.logits, "head_logits": out.head_logits, "n_accept": out.n_accept, "tokens": out.tokens}
    if c["kind"] == "prefill":
        st.kv.set_len([0] * c["batch"])
        sd.prefill(st.model, st.kv, st.tokens, st.lens)
        return [st.kv.read_rows(c["layers"] - 1, b, 0, n) for b, n in enumerate(st.lens)]
    if c["kind"] == "rows":
        for l in range(c["layers"]):
            for b in range(c["batch"]):
                st.kv.write_rows(l, b, 0, *st.rows[l][b])
        st.kv.set_len(st.lens)
        return [st.kv.read_rows(l, b, 0, n) for l in range(c["layers"]) for b, n in enumerate(st.lens)]
    n_acc, n_raw, tokens, slots, stats = sd.verify_tree_typical(st.tree, st.tok, st.logits, st.stop, temperature=0.8,
                                                                epsilon=0.09, delta=0.3)
    drawn = sd.sample_tokens(st.logits.view(-1, c["vocab"]), st.last, st.u, 0.8)
    return {"stats": stats, "n_accept": n_acc, "n_raw": n_raw, "tokens": tokens, "slots": slots, "drawn": drawn}


def prepare_accept(c, seed, st):
    """Logits as a trained model gives them (a few likely tokens per row), half of the nodes carrying a likely one."""
    B, T, V = c["batch"], c["nodes"], c["vocab"]
    g = gen(seed, 1)
    parent, depth, rank = tree_of(T, c["heads"], 10)
    T = len(parent)
    st.tree = sd.Tree(parent, depth, rank, c["heads"], 10)
    st.logits = torch.randn((B, T, V), generator=g, device=DEV) * 1.5
    st.tok = torch.randint(0, V, (B, T), generator=g, device=DEV, dtype=torch.int32)
    lift = torch.where(torch.rand((B, T), generator=g, device=DEV) < 0.5, 9.0, 0.0)
    for j in range(1, T):
        at = st.tok[:, j].long()
        st.logits[torch.arange(B, device=DEV), parent[j], at] += lift[:, j]
    st.stop = stop_words(V, seed)
    st.last = (torch.arange(B, device=DEV, dtype=torch.int32) * T + torch.randint(0, T, (B,), generator=g, device=DEV)).to(torch.int32)
    st.u = torch.rand(B, generator=g, device=DEV)
    return st


# --------------------------------------------------------------------------------------------- what a pass cannot avoid
def work(case):
    c = case
    if c["kind"] == "accept":
        n = c["batch"] * c["nodes"] * c["vocab"]
        return {"bytes": 4.0 * n + 8.0 * c["batch"] * c["nodes"], "flops": 6.0 * n}
    s = shape_of(c)
    size = 2 if s.dtype == "bf16" else 4
    d, F, V, L, B = s.d_model, s.d_ffn, s.vocab, s.n_layers, c["batch"]
    mean = 0.5 * (c["rows_lo"] + c["rows_hi"])
    if c["kind"] == "rows":
        return {"bytes": 4.0 * L * B * mean * 2 * d * size, "flops": 0.0}
    layer = 4.0 * d * d + 3.0 * d * F
    heads = float(s.n_medusa) * d * d
    if c["kind"] == "prefill":
        n = B * mean
        return {"bytes": size * (L * layer + V * d + heads) + 2.0 * L * n * d * size,
                "flops": 2.0 * n * L * layer + 2.0 * L * B * mean * mean * d + 2.0 * B * ((1 + s.n_medusa) * V * d + heads)}
    rows = B * c["nodes"]
    return {"bytes": size * (L * layer + V * d + heads + 2.0 * L * B * mean * d) + 4.0 * V * (rows + B * s.n_medusa),
            "flops": 2.0 * rows * (L * layer + V * d) + 4.0 * L * rows * mean * d + 2.0 * B * (s.n_medusa * V * d + heads)}


def tolerance(case):
    """About four times what the path differs by from the same pass in 64 bits (exact, below). Keys and values are stored in
    16 bits: two correct evaluations round some of them to different neighbours, which is all that the bfloat16 cases
    show, a little more of it per layer."""
    if case["kind"] == "rows":
        return "exact"
    if case["kind"] == "accept":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}       # float32 sums of 64-bit precision across the row: 5e-8 seen
    if case["width"] == "tiny":
        return {"rel": 4e-6, "max": 1e-4}                      # float32 throughout: 8e-7 seen
    if case["kind"] == "prefill":
        return {"rel": 5e-3, "max": 0.05}                      # bfloat16 rows themselves: 1.3e-3 seen
    return {"rel": 2e-3, "max": 0.05}                          # logits: 2e-5 to 5e-4 seen


# --------------------------------------------------------------------------------------------- the same in 64 bits
def exact(case, seed):
    c = case
    if c["kind"] == "accept":
        return exact_accept(c, seed)
    s = shape_of(c)
    lens = lengths(c)
    if c["kind"] == "rows":
        return [cache_rows(s, seed, l, b, n) for l in range(s.n_layers) for b, n in enumerate(lens)]
    if c["kind"] == "prefill":
        tokens = torch.randint(0, s.vocab, (sum(lens),), generator=gen(seed, 20002), device=DEV, dtype=torch.int32).split(lens)
        pos = [torch.arange(n, device=DEV) for n in lens]
        vis = [torch.ones((n, n), dtype=torch.bool, device=DEV).tril() for n in lens]
        return forward(s, seed, tokens, pos, vis, [0] * len(lens), last_kv=True)
    root, cand = drafts(s, c, seed)
    parent, depth, rank = tree_of(c["nodes"], s.n_medusa, s.topk)
    T = len(parent)
    anc = torch.zeros((T, T), dtype=torch.bool, device=DEV)
    for j in range(T):
        anc[j, j] = True
        if j:
            anc[j] |= anc[parent[j]]
    tokens = [torch.stack([root[b]] + [cand[b, depth[j] - 1, rank[j]] for j in range(1, T)]) for b in range(c["batch"])]
    pos = [n + torch.tensor(depth, device=DEV) for n in lens]
    h = forward(s, seed, tokens, pos, [anc] * c["batch"], lens)
    lm = weight(s, seed, "lm_head").double().T
    logits = torch.stack([x @ lm for x in h])
    # the last kept node: along the deepest path whose tokens are the arg-max at their parents, cut at the last stop token
    stop = stop_words(s.vocab, seed).long()
    kept = []
    for b in range(c["batch"]):
        am = logits[b].argmax(-1).tolist()
        tok = tokens[b].tolist()
        ok = [True] + [False] * (T - 1)
        for j in range(1, T):
            ok[j] = ok[parent[j]] and tok[j] == am[parent[j]]
        j = max((j for j in range(T) if ok[j]), key=lambda j: (depth[j], -j))
        chain = [j]
        while parent[chain[-1]] >= 0:
            chain.append(parent[chain[-1]])
        chain.reverse()
        ends = [i for i, n in enumerate(chain) if int(stop[tok[n] // 32]) >> (tok[n] % 32) & 1]
        kept.append(chain[ends[-1]] if ends and c["nodes"] > 1 else chain[-1])
    last = torch.stack([h[b][kept[b]] for b in range(c["batch"])])
    head = []
    for i in range(s.n_medusa):
        z = last @ weight(s, seed, "medusa%d.w" % i).double().T + weight(s, seed, "medusa%d.b" % i).double()
        head.append((last + z * torch.sigmoid(z)) @ lm)
    return {"logits": logits, "head_logits": torch.stack(head, 1), "n_accept": None, "tokens": None}


def forward(s, seed, tokens, pos, vis, n_cache, last_kv=False):
    """Final-norm rows of every sequence (last_kv: the last layer's keys and values instead), in 64 bits; keys and values are
    numbers of the storage type, as the framework defines a model's dtype."""
    B, nh, hd, d = len(tokens), s.n_heads, s.head_dim, s.d_model
    dt = dtype_of(s)

    def norm(x):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + s.rms_eps)

    def stored(x):
        return x.to(dt).double() if s.dtype == "bf16" else x

    def rotate(x, p):
        f = s.rope_theta ** (-2.0 * torch.arange(hd // 2, device=DEV, dtype=torch.float64) / hd)
        a = p.double()[:, None, None] * f
        co, si, x1, x2 = a.cos(), a.sin(), x[..., : hd // 2], x[..., hd // 2:]
        return torch.cat([x1 * co - x2 * si, x2 * co + x1 * si], -1)

    emb = weight(s, seed, "embed")
    x = [emb[t.long()].double() for t in tokens]
    del emb
    for l in range(s.n_layers):
        w = {k: weight(s, seed, "l%d.%s" % (l, k)).double().T for k in ("wqkv", "wo")}
        rows = []
        for b in range(B):
            q, k, v = (norm(x[b]) @ w["wqkv"]).view(-1, 3, nh, hd).unbind(1)
            q, k, v = rotate(q, pos[b]), stored(rotate(k, pos[b])), stored(v)
            if last_kv and l == s.n_layers - 1:
                rows.append((k, v))
                continue
            n, m = n_cache[b], len(tokens[b])
            if n:
                kc, vc = cache_rows(s, seed, l, b, n)
                k, v = torch.cat([kc.double(), k]), torch.cat([vc.double(), v])
            seen = torch.cat([torch.ones((m, n), dtype=torch.bool, device=DEV), vis[b]], 1)
            o = torch.empty_like(q)
            for h in range(nh):
                sc = (q[:, h].contiguous() @ k[:, h].contiguous().T) / math.sqrt(hd)
                o[:, h] = torch.softmax(sc.masked_fill(~seen, -math.inf), -1) @ v[:, h].contiguous()
            x[b] = x[b] + o.reshape(m, d) @ w["wo"]
        if rows:
            return rows
        del w
        w = {k: weight(s, seed, "l%d.%s" % (l, k)).double().T for k in ("w_gate", "w_up", "w_down")}
        for b in range(B):
            f = norm(x[b])
            g = f @ w["w_gate"]
            x[b] = x[b] + (g * torch.sigmoid(g) * (f @ w["w_up"])) @ w["w_down"]
        del w
    return [norm(y) for y in x]


def exact_accept(c, seed):
    """The rows' statistics at the temperature; the whole numbers that follow from them have no value here."""
    st = prepare_accept(c, seed, State())
    x = st.logits.double() / 0.8
    mx = x.max(-1, keepdim=True).values
    e = torch.exp(x - mx)
    z = e.sum(-1)
    ent = torch.log(z) - (e * (x - mx)).sum(-1) / z
    thr = torch.minimum(torch.full_like(ent, math.log(0.09)), math.log(0.3) - ent)
    stats = torch.stack([mx[..., 0] * 0.8, z, ent, thr + torch.log(z)], -1)
    return {"stats": stats, "n_accept": None, "n_raw": None, "tokens": None, "slots": None, "drawn": None}
