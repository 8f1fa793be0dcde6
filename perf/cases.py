"""The work that a user of liblsv has it do, as cases that can be timed and compared.

One speculative round is select -> verify -> accept (-> commit).  Almost all of its time is the
verify forward pass, so most cases are that pass through lsv_verify_block / lsv_verify_tree /
lsv_verify_paged: decoder layers of the widths that the workloads of this repository use, from
one draft block of one sequence to a 512-row prefill chunk, over slab and paged caches.  The
cases of real width carry a few layers (every layer does the same work; bf16 rounding drifts with
depth), one is a whole model.  The others are the calls around it, on the inputs that the
verify pass hands them.  Values come from the seed; sizes, context lengths and rows per sequence
are the case's own.
"""
import heapq
import math

import numpy as np
import torch

from paper_2608_08721_amd import decode, lsv, runtime

EPS, ROPE_BASE = 1e-5, 10000.0

# d_model, query heads, kv heads, head_dim, d_ff, vocabulary, dtype
SHAPES = {
    "llama3-8b": (4096, 32, 8, 128, 14336, 128256, "bf16"),
    "qwen2.5-32b": (5120, 40, 8, 128, 27648, 152064, "bf16"),
    "llama3-70b": (8192, 64, 8, 128, 28672, 128256, "bf16"),
    "small-bf16-hd128": (1024, 8, 2, 128, 2816, 4096, "bf16"),
    "tiny-bf16-gqa": (256, 4, 2, 64, 688, 1024, "bf16"),
    "tiny-f32": (256, 4, 4, 64, 688, 1024, "f32"),
}


class Shape:
    """A model's sizes under the names that runtime.model_config reads."""

    def __init__(self, model, layers):
        (self.d_model, self.n_q_heads, self.n_kv_heads, self.head_dim, self.d_ff, self.vocab,
         self.dtype) = SHAPES[model]
        self.n_layers, self.rms_eps, self.rope_base = layers, EPS, ROPE_BASE
        self.torch_dtype = torch.bfloat16 if self.dtype == "bf16" else torch.float32
        self.es = 2 if self.dtype == "bf16" else 4

    def layer_params(self):
        d, hd = self.d_model, self.head_dim
        return d * (self.n_q_heads + 2 * self.n_kv_heads) * hd + self.n_q_heads * hd * d + 3 * d * self.d_ff

    def params(self):
        return self.n_layers * self.layer_params() + self.d_model * self.vocab


def listed():
    return [
        # the selection of a small batch's lengths and the block that follows: the smallest call
        dict(name="select-joint-b16-g32", kind="select", mode="joint", batch=16, G=32),
        # greedy acceptance of the 70B workload's block under its row bound
        dict(name="accept-greedy-b4", kind="accept", mode="greedy", model="llama3-70b", batch=4, rows_lo=4, rows_hi=4,
             width=33),
        # speculative rejection sampling at temperature 1 over the largest vocabulary
        dict(name="accept-sample-b4", kind="accept", mode="sample", model="qwen2.5-32b", batch=4, rows_lo=7,
             rows_hi=11, width=17),
        # acceptance of a 512-node draft tree and the commit of its path in a whole model's cache
        dict(name="accept-tree-512", kind="tree-accept", model="llama3-8b", layers=32, batch=1, ctx=2048, nodes=512,
             depth=24),
        # a whole decoding round of the fp32 model, replayed as its captured graph: launch-bound
        dict(name="round-tiny-f32", kind="round", model="tiny-f32", layers=2, batch=1, ctx=128, G=16),
        # one sequence of an 8B model (half its depth, so that rounding has not drifted past what a
        # comparison can hold): the latency of interactive decoding
        dict(name="verify-8b-b1", kind="verify", model="llama3-8b", layers=16, batch=1, ctx_lo=2048, ctx_hi=2048,
             rows_lo=9, rows_hi=9, bound=17, cache="slab"),
        # the 70B workload: four sequences of 8K context, three drafts each, under the bound of 32 drafts
        dict(name="verify-70b-b4-g3", kind="verify", model="llama3-70b", layers=3, batch=4, ctx_lo=8192, ctx_hi=8192,
             rows_lo=4, rows_hi=4, bound=132, cache="slab"),
        # the 32B workload's longer blocks: more rows than one matrix-core tile
        dict(name="verify-32b-b4-g8", kind="verify", model="qwen2.5-32b", layers=4, batch=4, ctx_lo=4096, ctx_hi=4096,
             rows_lo=8, rows_hi=11, bound=68, cache="slab"),
        # a batch of ragged contexts with every draft verified: 264 rows
        dict(name="verify-8b-b8-g32", kind="verify", model="llama3-8b", layers=6, batch=8, ctx_lo=1024, ctx_hi=8192,
             rows_lo=33, rows_hi=33, bound=264, cache="slab"),
        # serving: many sequences of short blocks over a paged cache
        dict(name="verify-paged-b32", kind="verify", model="llama3-8b", layers=6, batch=32, ctx_lo=200, ctx_hi=4000,
             rows_lo=1, rows_hi=6, bound=192, cache="paged"),
        # a 512-node draft tree in one pass
        dict(name="verify-tree-512", kind="tree-verify", model="llama3-8b", layers=6, batch=1, ctx=2048, nodes=512,
             depth=24),
        # a 512-row prefill chunk behind 1.5K cached positions: the largest call
        dict(name="prefill-8b-512", kind="verify", model="llama3-8b", layers=6, batch=1, ctx_lo=1536, ctx_hi=1536,
             rows_lo=512, rows_hi=512, bound=512, cache="slab"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["verify"] * 9 + ["tree-verify", "select", "accept", "accept", "tree-accept", "round"])
    big = ["llama3-8b", "llama3-8b", "qwen2.5-32b", "llama3-70b"]
    if kind == "select":
        return dict(kind=kind, mode=rng.choice(["joint", "marginal", "exhaustive", "alg1"]), batch=_log(rng, 1, 64),
                    G=rng.randint(4, 64))
    if kind == "accept":
        batch = _log(rng, 1, 16)
        width = rng.randint(2, min(33, 256 // batch))
        lo = rng.randint(1, width)
        return dict(kind=kind, mode=rng.choice(["greedy", "sample"]), model=rng.choice(big + ["small-bf16-hd128"]),
                    batch=batch, rows_lo=lo, rows_hi=rng.randint(lo, width), width=width)
    if kind == "round":
        return dict(kind=kind, model="tiny-f32", layers=rng.randint(1, 3), batch=_log(rng, 1, 4),
                    ctx=_log(rng, 32, 1000), G=rng.randint(3, 24))
    if kind in ("tree-verify", "tree-accept"):
        model = rng.choice(["llama3-8b", "qwen2.5-32b"])
        batch = rng.choice([1, 1, 2, 4])
        nodes = _log(rng, 24, 512 // batch)
        layers = rng.randint(1, 3) if kind == "tree-verify" else rng.choice([16, 32])
        return dict(kind=kind, model=model, layers=layers, batch=batch, ctx=_log(rng, 256, 4096), nodes=nodes,
                    depth=rng.randint(6, 32))
    model = rng.choice(big + ["small-bf16-hd128", "tiny-bf16-gqa", "tiny-f32"])
    tiny = model not in big
    batch = _log(rng, 1, 8 if tiny else 64)
    most = 64 if tiny else 272 if model != "llama3-8b" else 512
    per = max(1, most // batch)
    rows_hi = _log(rng, 1, per)
    rows_lo = rng.randint(max(1, rows_hi // 2), rows_hi)
    bound = rng.choice([rows_hi * batch, min(most, rows_hi * batch + rng.randint(0, 3 * batch))])
    ctx_hi = _log(rng, 64, 1024 if tiny else min(8192, 65536 // batch))
    ctx_lo = rng.randint(1, ctx_hi)
    layers = rng.randint(1, 3 if tiny else {"llama3-8b": 4, "qwen2.5-32b": 3, "llama3-70b": 2}[model])
    return dict(kind="verify", model=model, layers=layers, batch=batch, ctx_lo=ctx_lo, ctx_hi=ctx_hi, rows_lo=rows_lo,
                rows_hi=rows_hi, bound=bound, cache=rng.choice(["slab", "slab", "paged"]))


# ------------------------------------------------------------------ sizes of a case
def _spread(lo, hi, n, step):
    """n whole numbers from lo to hi, evenly spaced, in an order that is not sorted."""
    v = [lo + (hi - lo) * i // max(1, n - 1) for i in range(n)] if n > 1 else [hi]
    while math.gcd(step, n) != 1:
        step += 1
    return [v[(i * step) % n] for i in range(n)]


def _rows(case):
    if case["kind"].startswith("tree"):
        return [case["nodes"]] * case["batch"]
    return _spread(case["rows_lo"], case["rows_hi"], case["batch"], 3)


def _contexts(case):
    if "ctx" in case:
        return [case["ctx"]] * case["batch"]
    return _spread(case["ctx_lo"], case["ctx_hi"], case["batch"], 5)


def _offsets(rows):
    return [0] + [int(x) for x in np.cumsum(rows)]


# ------------------------------------------------------------------ seeded values
def _gen(seed, stream, device="cuda"):
    return torch.Generator(device=device).manual_seed((int(seed) * 1000003 + stream * 7919 + 17) % (1 << 62))


def _normal(g, shape, std, dtype):
    return torch.randn(shape, generator=g, device="cuda", dtype=dtype).mul_(std)


def _layer_weights(s, seed, layer):
    """One layer's matrices [out, in] and norm gains, as a checkpoint of this shape holds them."""
    g, d, hd, F, t = _gen(seed, 100 + layer), s.d_model, s.head_dim, s.d_ff, s.torch_dtype
    q, kv = s.n_q_heads * hd, s.n_kv_heads * hd
    w = [_normal(g, shp, 0.02, t) for shp in ((q, d), (kv, d), (kv, d), (d, q), (F, d), (F, d), (d, F))]
    return w + [torch.rand(d, generator=g, device="cuda").add_(0.5).to(t) for _ in range(2)]


def _global_weights(s, seed):
    g, t = _gen(seed, 1), s.torch_dtype
    embed = _normal(g, (s.vocab, s.d_model), 0.02, t)
    gain = torch.rand(s.d_model, generator=g, device="cuda").add_(0.5).to(t)
    return embed, gain, _normal(g, (s.vocab, s.d_model), 0.02, t)


def _context_kv(s, seed, layer, b, C):
    """Cached K and V of one layer and sequence, [kv head][position][head_dim]."""
    g = _gen(seed, 10000 + 100 * layer + b)
    return [_normal(g, (s.n_kv_heads, C, s.head_dim), 1.0, s.torch_dtype) for _ in range(2)]


def _tokens(s, seed, n):
    return torch.randint(0, s.vocab, (n,), generator=_gen(seed, 2), device="cuda", dtype=torch.int32)


def _tree(case, seed):
    """Parents of each sequence's draft tree: the most probable prefixes, best first, of a few
    candidates per depth (what a tree drafter keeps under a node budget)."""
    out = []
    for b in range(case["batch"]):
        rng = np.random.default_rng([int(seed), b, 77])
        prob = [np.sort(rng.dirichlet(np.full(8, 0.5)))[::-1] for _ in range(case["depth"])]
        parents, depths, heap = [-1], [0], [(-prob[0][j], 0, 0, j) for j in range(8)]
        while len(parents) < case["nodes"]:
            neg, par, d, j = heapq.heappop(heap)
            node = len(parents)
            parents.append(par)
            depths.append(d + 1)
            if d + 1 < case["depth"]:
                for jj in range(8):
                    heapq.heappush(heap, (neg * prob[d + 1][jj], node, d + 1, jj))
        out.append((parents, depths))
    return out


def _i32(x):
    return torch.tensor(x, dtype=torch.int32, device="cuda")


def _model(s, seed):
    cfg = runtime.model_config(s)
    dm = runtime.DeviceModel(cfg)
    lsv.lsv_pack_globals(cfg, *_global_weights(s, seed), dm.buf)
    for l in range(s.n_layers):
        lsv.lsv_pack_layer(cfg, l, *_layer_weights(s, seed, l), dm.buf)
    torch.cuda.synchronize()
    return cfg, dm


def _cache(s, cfg, case, seed, contexts, rows):
    """The KV cache with its context in place, and its capacity in positions per sequence."""
    B, need = case["batch"], max(c + r for c, r in zip(contexts, rows))
    cap = runtime.kv_capacity(need)
    if case.get("cache") == "paged":
        per = cap // lsv.LSV_KV_PAGE
        order = np.random.default_rng([int(seed), 5]).permutation(B * per)
        kv = runtime.PagedKVCache(cfg, B * per, order.reshape(B, per))
    else:
        kv = runtime.KVCache(cfg, B, cap)
    for l in range(s.n_layers):
        for b in range(B):
            kv.write(l, b, 0, *_context_kv(s, seed, l, b, contexts[b]))
    return kv, cap


# ------------------------------------------------------------------ the cases' states
def prepare(case, seed):
    return {"select": _prepare_select, "accept": _prepare_accept, "tree-accept": _prepare_tree_accept,
            "round": _prepare_round}.get(case["kind"], _prepare_verify)(case, seed)


def _prepare_verify(case, seed):
    s = Shape(case["model"], case["layers"])
    rows, ctx = _rows(case), _contexts(case)
    cfg, dm = _model(s, seed)
    kv, cap = _cache(s, cfg, case, seed, ctx, rows)
    B, M = case["batch"], sum(rows)
    bound = case.get("bound", M)
    ws = runtime.Workspace(lsv.lsv_verify_workspace_bytes(cfg, B, bound, cap))
    st = dict(case=case, cfg=cfg, dm=dm, kv=kv, cap=cap, ws=ws, M=M, bound=bound, batch=B, seq_len=_i32(ctx),
              tokens=torch.zeros(bound, dtype=torch.int32, device="cuda"), offsets=_i32(_offsets(rows)),
              logits=torch.zeros((bound, s.vocab), dtype=torch.float32, device="cuda"),
              status=torch.zeros(B, dtype=torch.int32, device="cuda"), parents=None)
    st["tokens"][:M] = _tokens(s, seed, M)
    if case["kind"] == "tree-verify":
        st["parents"] = _i32([p for parents, _ in _tree(case, seed) for p in parents])
    return st


def _accept_inputs(s, seed, rows, share):
    """Logits of every block row and tokens that a fair share of drafts agree with."""
    M = sum(rows)
    g = _gen(seed, 3)
    logits = torch.randn((M, s.vocab), generator=g, device="cuda").mul_(2.0)
    tokens = torch.randint(0, s.vocab, (M,), generator=g, device="cuda", dtype=torch.int32)
    hit = torch.rand(M, generator=g, device="cuda") < share
    return logits, tokens, hit


def _prepare_accept(case, seed):
    s = Shape(case["model"], 1)
    B, rows, width = case["batch"], _rows(case), case["width"]
    off, M, bound = _offsets(rows), sum(rows), case["batch"] * case["width"]
    data, tokens, hit = _accept_inputs(s, seed, rows, 0.8)
    logits = torch.zeros((bound, s.vocab), device="cuda")
    logits[:M] = data
    probs = None
    if case["mode"] == "sample":
        # proposals near the target's own distribution, as a trained drafter's are
        keep = torch.ones(M, dtype=torch.bool)
        keep[[o - 1 for o in off[1:]]] = False  # row v - 1 scores draft v: the last row scores none
        rows_of = torch.nonzero(keep).flatten().cuda()
        if len(rows_of):
            z = data[rows_of] + 0.5 * torch.randn((len(rows_of), s.vocab), generator=_gen(seed, 4), device="cuda")
            probs = torch.softmax(z, dim=1)
            # drawn by the exponential race, so that the draw does not depend on the order of a sum
            u = torch.rand(probs.shape, generator=_gen(seed, 5), device="cuda").clamp_(min=1e-30)
            tokens[rows_of + 1] = torch.argmin(-torch.log(u) / probs, dim=1).to(torch.int32)
        else:
            probs = torch.zeros((1, s.vocab), device="cuda")
    else:
        top = torch.argmax(data, dim=1).to(torch.int32)
        tokens[1:] = torch.where(hit[1:], top[:-1], tokens[1:])
    padded = torch.zeros(bound, dtype=torch.int32, device="cuda")
    padded[:M] = tokens
    ctx = _i32([1024 + 7 * b for b in range(B)])
    return dict(case=case, batch=B, vocab=s.vocab, logits=logits, offsets=_i32(off), bound=bound, width=width,
                tokens=padded, probs=probs, seed=int(seed) & 0xFFFF, start=ctx, seq_len=ctx.clone(),
                acc=torch.zeros(B, dtype=torch.int32, device="cuda"),
                out=torch.zeros((B, width), dtype=torch.int32, device="cuda"),
                roots=torch.zeros(B, dtype=torch.int32, device="cuda"),
                status=torch.zeros(B, dtype=torch.int32, device="cuda"),
                ws=runtime.Workspace(lsv.lsv_accept_workspace_bytes(B, bound, s.vocab)))


def _prepare_tree_accept(case, seed):
    s = Shape(case["model"], case["layers"])
    B, rows, C = case["batch"], _rows(case), case["ctx"]
    M, width = sum(rows), lsv.LSV_MAX_SEQ_ROWS
    logits, tokens, _ = _accept_inputs(s, seed, rows, 0.0)
    parents = [p for p, _ in _tree(case, seed)]
    top = torch.argmax(logits, dim=1).cpu().tolist()
    tok = tokens.cpu().tolist()
    rng = np.random.default_rng([int(seed), 6])
    for b, par in enumerate(parents):  # one child in two of every node carries its parent's argmax
        for i in range(1, len(par)):
            if rng.random() < 0.5:
                tok[b * case["nodes"] + i] = top[b * case["nodes"] + par[i]]
    cfg = runtime.model_config(s)
    kv = runtime.KVCache(cfg, B, runtime.kv_capacity(C + case["nodes"]))
    g = _gen(seed, 8)  # the verify pass left every node's K and V at its slot
    blocks = kv.buf.view(s.torch_dtype).view(s.n_layers, -1)
    for l in range(s.n_layers):
        blocks[l].normal_(0.0, 1.0, generator=g)
    start = _i32([C] * B)
    return dict(case=case, batch=B, vocab=s.vocab, cfg=cfg, kv=kv, logits=logits, offsets=_i32(_offsets(rows)),
                parents=_i32([p for par in parents for p in par]), tokens=_i32(tok), M=M, width=width, start=start,
                seq_len=start.clone(), acc=torch.zeros(B, dtype=torch.int32, device="cuda"),
                out=torch.zeros((B, width), dtype=torch.int32, device="cuda"),
                path=torch.zeros((B, width), dtype=torch.int32, device="cuda"),
                status=torch.zeros(B, dtype=torch.int32, device="cuda"),
                ws=runtime.Workspace(lsv.lsv_accept_workspace_bytes(B, M, s.vocab)))


def _confidences(case, seed):
    rng = np.random.default_rng([int(seed), 9])
    return (rng.beta(6.0, 3.0, (case["batch"], case["G"])) * 0.9 ** np.arange(1, case["G"] + 1)).astype(np.float32)


def _costs(n):
    """A measured-looking verify cost: flat inside a 16-row tile, a step at each further one."""
    return [1.0 + 0.002 * r + 0.12 * (r // 16) for r in range(n)]


def _prepare_select(case, seed):
    B, G = case["batch"], case["G"]
    n = B * G + 1 if case["mode"] == "joint" else G + 1
    bound = min(lsv.LSV_MAX_ROWS, B * (G + 1))
    g = _gen(seed, 11)
    width = min(G, lsv.LSV_MAX_SEQ_ROWS - 1)
    return dict(case=case, batch=B, G=G, width=width, bound=bound,
                conf=torch.tensor(_confidences(case, seed), device="cuda"),
                cost=torch.tensor(_costs(n), dtype=torch.float64, device="cuda"),
                roots=torch.randint(0, 128256, (B,), generator=g, device="cuda", dtype=torch.int32),
                drafts=torch.randint(0, 128256, (B, width), generator=g, device="cuda", dtype=torch.int32),
                gamma=torch.zeros(B, dtype=torch.int32, device="cuda"),
                aux=torch.zeros(B, dtype=torch.int32, device="cuda"),
                total=torch.zeros(1, dtype=torch.int32, device="cuda"),
                offsets=torch.zeros(B + 1, dtype=torch.int32, device="cuda"),
                tokens=torch.zeros(bound, dtype=torch.int32, device="cuda"),
                status=torch.zeros(B, dtype=torch.int32, device="cuda"))


def _prepare_round(case, seed):
    s = Shape(case["model"], case["layers"])
    B, G, C = case["batch"], case["G"], case["ctx"]
    cfg, dm = _model(s, seed)
    kv, cap = _cache(s, cfg, case, seed, [C] * B, [G + 1] * B)
    loop = decode.DecodeLoop(cfg, dm, kv, cap, B, G, "marginal", None, cost=[1.0 + 0.05 * d for d in range(G + 1)])
    loop.conf.copy_(torch.tensor(_confidences(case, seed)))
    toks = _tokens(s, seed, B * (G + 1)).view(B, G + 1)
    loop.drafts.copy_(toks[:, 1:])
    st = dict(case=case, loop=loop, seq_len=_i32([C] * B), roots=toks[:, 0].contiguous())
    loop.reset(st["seq_len"], st["roots"])
    loop.round()  # warms the launches; the graph's rounds start from reset()
    torch.cuda.synchronize()
    loop.capture()
    return st


# ------------------------------------------------------------------ one pass
def run(st):
    return {"select": _run_select, "accept": _run_accept, "tree-accept": _run_tree_accept,
            "round": _run_round}.get(st["case"]["kind"], _run_verify)(st)


def _run_verify(st):
    kv, tail = st["kv"], (st["bound"], st["cap"], st["logits"], st["status"], st["ws"].buf, st["ws"].nbytes)
    head = (st["batch"], st["seq_len"], st["tokens"], st["offsets"])
    if isinstance(kv, runtime.PagedKVCache):
        lsv.lsv_verify_paged(st["cfg"], st["dm"].buf, kv.buf, kv.n_pages, kv.table, kv.max_pages, *head,
                             st["parents"], *tail)
    elif st["parents"] is not None:
        lsv.lsv_verify_tree(st["cfg"], st["dm"].buf, kv.buf, st["cap"], *head, st["parents"], *tail)
    else:
        lsv.lsv_verify_block(st["cfg"], st["dm"].buf, kv.buf, st["cap"], *head, *tail)
    return {"logits": st["logits"][:st["M"]], "status": st["status"],
            "kv": kv.buf.view(runtime.storage_dtype(st["cfg"]))}


def _run_accept(st):
    st["seq_len"].copy_(st["start"])
    sample = st["case"]["mode"] == "sample"
    lsv.lsv_accept(lsv.LSV_ACC_SAMPLE if sample else lsv.LSV_ACC_GREEDY, st["batch"], st["vocab"], st["logits"],
                   st["offsets"], st["bound"], st["width"], st["tokens"], st["probs"], 1.0 if sample else 0.0,
                   st["seed"], 3, st["acc"], st["out"], st["seq_len"], st["status"], st["ws"].buf, st["ws"].nbytes)
    lsv.lsv_next_roots(st["batch"], st["acc"], st["out"], st["width"], st["status"], st["roots"])
    return {k: st[k] for k in ("acc", "out", "seq_len", "status", "roots")}


def _run_tree_accept(st):
    st["seq_len"].copy_(st["start"])
    lsv.lsv_accept_tree(st["batch"], st["vocab"], st["logits"], st["offsets"], st["parents"], st["tokens"], st["M"],
                        st["width"], st["acc"], st["out"], st["path"], st["seq_len"], st["status"], st["ws"].buf,
                        st["ws"].nbytes)
    lsv.lsv_commit_tree(st["cfg"], st["kv"].buf, st["kv"].capacity, st["batch"], st["seq_len"], st["acc"], st["path"],
                        st["width"], st["status"])
    out = {k: st[k] for k in ("acc", "out", "path", "seq_len", "status")}
    out["kv"] = st["kv"].buf.view(runtime.storage_dtype(st["cfg"]))
    return out


def _run_select(st):
    B, G, mode = st["batch"], st["G"], st["case"]["mode"]
    if mode == "joint":
        lsv.lsv_select_joint(B, G, st["conf"], st["cost"], G, 0, st["gamma"], st["total"], st["offsets"], st["status"])
    else:
        m = {"marginal": lsv.LSV_SEL_MARGINAL, "exhaustive": lsv.LSV_SEL_EXHAUSTIVE, "alg1": lsv.LSV_SEL_ALG1}[mode]
        lsv.lsv_select_length(m, B, G, st["conf"], st["cost"], 1, G, 2.2, 8, 0, st["gamma"], st["aux"], st["offsets"],
                              st["status"])
    lsv.lsv_pack_block(B, st["width"], st["offsets"], st["bound"], st["roots"], st["drafts"], st["tokens"], None)
    return {k: st[k] for k in ("gamma", "aux", "total", "offsets", "tokens", "status")}


def _run_round(st):
    loop = st["loop"]
    loop.reset(st["seq_len"], st["roots"])
    loop.replay()
    return {"logits": loop.logits, "acc": loop.acc, "out": loop.out, "gamma": loop.gamma, "seq_len": loop.seq_len,
            "roots": loop.roots, "status": loop.status}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind == "select":
        B, G = case["batch"], case["G"]
        n = B * G + 1 if case["mode"] == "joint" else G + 1
        return {"bytes": 4.0 * B * G + 8.0 * n + 4.0 * B * 8, "flops": 3.0 * B * G + 2.0 * n}
    if kind in ("accept", "tree-accept"):
        V, M = SHAPES[case["model"]][5], sum(_rows(case))
        # sampling: one softmax pass over every row, then one draw per sequence over its row of p and of q
        sample = case.get("mode") == "sample"
        return {"bytes": 4.0 * V * (M + (2 * case["batch"] if sample else 0)), "flops": (4.0 if sample else 1.0) * M * V}
    s = Shape(case["model"], case["layers"])
    if kind == "round":
        rows, ctx = [case["G"] // 2 + 1] * case["batch"], [case["ctx"]] * case["batch"]
    else:
        rows, ctx = _rows(case), _contexts(case)
    M = sum(rows)
    kv_row = 2.0 * s.n_kv_heads * s.head_dim * s.es * s.n_layers
    return {"bytes": s.params() * s.es + kv_row * (sum(ctx) + M) + 4.0 * M * s.vocab + s.es * M * s.d_model,
            "flops": 2.0 * M * s.params() + 4.0 * s.n_layers * s.n_q_heads * s.head_dim
            * sum(r * (c + (r + 1) / 2) for r, c in zip(rows, ctx))}


def tolerance(case):
    # Whole numbers, and the commit's copies, are exact.  fp32 logits differ by the order of 32-bit
    # sums (7e-7 off 64 bits).  A bf16 model rounds its operands to 8 bits at every projection: a
    # sum taken in another order moves some of them by one unit, which the layers behind carry on.
    # Measured between two orders (another k split of the products, other attention splits): 7e-3 to
    # 1.1e-2 at 4 to 6 layers, the largest single difference 0.07; four times that is over 3e-2.
    if case["kind"] in ("select", "accept", "tree-accept"):
        return "exact"
    if SHAPES[case["model"]][6] == "f32":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}
    return {"rel": 0.03, "max": 0.3, "differ": 0.0}


# ------------------------------------------------------------------ the same in 64 bits
def exact(case, seed):
    """The verify pass in float64 torch; whole-number outputs are compared as they are."""
    if case["kind"] == "round":
        return _exact_round(case, seed)
    if case["kind"] not in ("verify", "tree-verify"):
        return None
    rows, ctx = _rows(case), _contexts(case)
    parents = [p for p, _ in _tree(case, seed)] if case["kind"] == "tree-verify" else None
    s = Shape(case["model"], case["layers"])
    return {"logits": _forward64(s, seed, _tokens(s, seed, sum(rows)).long(), rows, ctx, parents), "status": None,
            "kv": None}


def _forward64(s, seed, tokens, rows, ctx, parents=None):
    def R(x):  # the model dtype's rounding where an operand or the cache is stored
        return x.to(s.torch_dtype).double()

    def norm(x, g):
        return R(x / torch.sqrt(x.square().mean(1, keepdim=True) + EPS) * g.double())

    def linear(x, w):
        return torch.cat([x @ part.double().T for part in w.split(16384)], dim=1)

    def rope(x, pos):
        half = s.head_dim // 2
        i = torch.arange(half, device="cuda", dtype=torch.float64)
        a = pos.double()[:, None] * ROPE_BASE ** (-2.0 * i / s.head_dim)[None, :]
        c, sn = torch.cos(a)[:, None, :], torch.sin(a)[:, None, :]
        return torch.cat([x[..., :half] * c - x[..., half:] * sn, x[..., half:] * c + x[..., :half] * sn], dim=-1)

    off, hd, group = _offsets(rows), s.head_dim, s.n_q_heads // s.n_kv_heads
    pos, masks = [], []
    for b, (n, C) in enumerate(zip(rows, ctx)):
        par = list(range(-1, n - 1)) if parents is None else parents[b]
        depth, vis = [0] * n, torch.zeros((n, n), dtype=torch.bool)
        for i in range(n):
            if i:
                depth[i] = depth[par[i]] + 1
                vis[i] = vis[par[i]]
            vis[i, i] = True
        pos += [C + d for d in depth]
        masks.append(torch.cat([torch.ones((n, C), dtype=torch.bool), vis], dim=1).cuda())
    pos = torch.tensor(pos, device="cuda")
    embed, final, head = _global_weights(s, seed)
    h = embed[tokens].double()
    for l in range(s.n_layers):
        wq, wk, wv, wo, wg, wu, wd, g1, g2 = _layer_weights(s, seed, l)
        a, M = norm(h, g1), len(tokens)
        q = R(rope(linear(a, wq).view(M, -1, hd), pos))
        k = R(rope(linear(a, wk).view(M, -1, hd), pos))
        v = R(linear(a, wv)).view(M, -1, hd)
        o = torch.zeros((M, s.n_q_heads, hd), dtype=torch.float64, device="cuda")
        for b, C in enumerate(ctx):
            r = slice(off[b], off[b + 1])
            kc, vc = _context_kv(s, seed, l, b, C)
            K = torch.cat([kc.double(), k[r].transpose(0, 1)], dim=1)
            V = torch.cat([vc.double(), v[r].transpose(0, 1)], dim=1)
            for hq in range(s.n_q_heads):
                sc = (q[r, hq] @ K[hq // group].T) / math.sqrt(hd)
                o[r, hq] = torch.softmax(sc.masked_fill(~masks[b], -math.inf), dim=1) @ V[hq // group]
        h = h + linear(R(o.reshape(M, -1)), wo)
        a = norm(h, g2)
        gate = linear(a, wg)
        h = h + linear(R(gate / (1.0 + torch.exp(-gate)) * linear(a, wu)), wd)
    return linear(norm(h, final), head)


def _exact_round(case, seed):
    s = Shape(case["model"], case["layers"])
    B, G, C = case["batch"], case["G"], case["ctx"]
    gammas = []
    for q in _confidences(case, seed).astype(np.float64):
        f = np.cumsum(np.cumprod(q)) / (1.0 + 0.05 * np.arange(1, G + 1))
        d = 1
        while d < G and f[d] > f[d - 1]:
            d += 1
        gammas.append(d)
    toks = _tokens(s, seed, B * (G + 1)).view(B, G + 1).long()
    rows = [g + 1 for g in gammas]
    lg = _forward64(s, seed, torch.cat([toks[b, :rows[b]] for b in range(B)]), rows, [C] * B)
    full = torch.zeros((B * (G + 1), s.vocab), dtype=torch.float64, device="cuda")
    full[:sum(rows)] = lg
    return {"logits": full, "acc": None, "out": None, "gamma": None, "seq_len": None, "roots": None, "status": None}
