"""The work a decoding server has this library do, as cases that can be timed and compared.

A case is a dict of plain numbers and texts. Five kinds:

  layer    evict_verify_layer: one pass of the draft-tree nodes of `trees` sequences through one decoder layer;
           with `step` also the prefix selection before it and the greedy acceptance after it (the default
           benchmark's step).
  iterate  selection, compaction, a stack of layers on paged caches and the LM head's score rows, with the
           selected length read on the device (evict_dynamic_tokens): a speculative iteration up to acceptance.
  lm       the LM head over the verified nodes: score rows, or arg max with greedy acceptance.
  accept   acceptance under sampling on given score rows and the commit of the accepted rows to the caches.
  select   prefix selection of a batch of trees and the gather of the kept rows.

Inputs follow the statistics of the repository's own generators: weights N(0, 0.02), keys and values N(0, 1),
hidden states correlated along the branches of the tree (child = parent + noise * N(0, 1)), draft probabilities
uniform on (0.05, 1).
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2605_00342_amd as ev
from paper_2605_00342_amd import harness

DEV = "cuda:0"
VOCAB = 151936

# The repository's own model shapes.
MODELS = {
    "tiny": dict(dtype="f32", d=256, Hq=4, Hkv=2, D=64, E=16, k=2, F=128, theta=1e4),
    "qwen3": dict(dtype="bf16", d=2048, Hq=32, Hkv=4, D=128, E=128, k=8, F=768),
    "dsv2lite": dict(dtype="bf16", d=2048, Hq=16, Hkv=16, D=128, E=64, k=6, F=1408, n_shared=2, theta=1e4),
    "qwen3_235b_tp8": dict(dtype="bf16", d=4096, Hq=8, Hkv=1, D=128, E=128, k=8, F=192),
    "ling_flash2_tp4": dict(dtype="bf16", d=4096, Hq=8, Hkv=1, D=128, E=256, k=8, F=256, n_shared=1, router_norm="sigmoid"),
}
# Tokens routed alike because they share a branch: the union of N nodes is that of about N ** SPREAD independent tokens
# (fitted to the unions measured for these trees at 32 to 128 nodes).
SPREAD = {0.2: 0.22, 0.5: 0.48, 1.0: 0.63}


def cfg_of(case, **more):
    m = dict(n_shared=0, eps=1e-6, theta=1e6, router_norm="softmax", name=case["model"])
    m.update(MODELS[case["model"]])
    m.update(more)
    return SimpleNamespace(**m)


def listed():
    return [
        # the smallest layer and the 32-bit path: eight nodes, every launch far below a microsecond of work
        {"name": "layer_f32_8", "kind": "layer", "model": "tiny", "trees": 1, "nodes": 8, "ctx": 64, "noise": 0.5},
        # plain autoregressive decoding of one sequence (a tree of one node), the reference every loop is compared with
        {"name": "layer_decode_1", "kind": "layer", "model": "qwen3", "trees": 1, "nodes": 1, "ctx": 2048, "noise": 0.5},
        # the default benchmark's step: select, verify a 32-node tree, accept
        {"name": "step_tree_32", "kind": "layer", "model": "qwen3", "trees": 1, "nodes": 32, "ctx": 2048, "noise": 0.5, "step": True},
        # the largest tree, widely spread branches, a longer context
        {"name": "layer_tree_128", "kind": "layer", "model": "qwen3", "trees": 1, "nodes": 128, "ctx": 4096, "noise": 1.0},
        # a small batch of sequences of different lengths
        {"name": "layer_batch_4x64", "kind": "layer", "model": "qwen3", "trees": 4, "nodes": 64, "ctx": 5555, "noise": 0.5},
        # the largest call a context of this model takes (8192 token-expert pairs): a loaded server
        {"name": "layer_batch_16x64", "kind": "layer", "model": "qwen3", "trees": 16, "nodes": 64, "ctx": 2048, "noise": 0.5},
        # many KV heads, shared experts, a long context
        {"name": "layer_mha_64_ctx8192", "kind": "layer", "model": "dsv2lite", "trees": 1, "nodes": 64, "ctx": 8192, "noise": 0.5},
        # one rank's share of a wide model: few heads, narrow experts, a long contraction
        {"name": "layer_wide_tp8_32", "kind": "layer", "model": "qwen3_235b_tp8", "trees": 1, "nodes": 32, "ctx": 2048, "noise": 0.5},
        # a whole iteration of the on-device loop over four layers and paged caches, returning the score rows
        {"name": "iterate_paged_41", "kind": "iterate", "model": "qwen3", "layers": 4, "nodes": 41, "ctx": 3000, "noise": 0.5, "page": 16},
        # the head of a greedy iteration
        {"name": "lm_greedy_32", "kind": "lm", "model": "qwen3", "trees": 1, "nodes": 32, "rows": False},
        # the tail of a sampling iteration of four sequences
        {"name": "accept_sampled_4x32", "kind": "accept", "trees": 4, "nodes": 32, "layers": 8, "cap": 512},
        # choosing what to verify for a batch
        {"name": "select_batch_16x64", "kind": "select", "model": "qwen3", "trees": 16, "nodes": 64},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "layer", "layer", "iterate", "lm", "accept", "select"])
    noise = rng.choice([0.2, 0.5, 0.5, 1.0])
    if kind == "layer":
        model = rng.choice(["qwen3", "qwen3", "qwen3", "dsv2lite", "qwen3_235b_tp8", "ling_flash2_tp4", "tiny"])
        trees = rng.choice([1, 1, 1, _log(rng, 2, 16)])
        nodes = _log(rng, 1, 128)
        most = {"qwen3": 1024, "tiny": 64}.get(model, 512)
        nodes = max(1, min(nodes, most // trees))
        room = {"qwen3": 32768, "dsv2lite": 16384, "tiny": 4096}.get(model, 32768)
        ctx = _log(rng, 17, max(32, min(room, 32768 // trees)))
        c = {"kind": "layer", "model": model, "trees": trees, "nodes": nodes, "ctx": ctx, "noise": noise}
        if rng.random() < 0.3:
            c["step"] = True
        return c
    if kind == "iterate":
        return {"kind": "iterate", "model": rng.choice(["qwen3", "ling_flash2_tp4"]), "layers": rng.randint(2, 4), "nodes": _log(rng, 4, 64),
                "ctx": _log(rng, 100, 8000), "noise": noise, "page": rng.choice([16, 64, 256])}
    if kind == "lm":
        return {"kind": "lm", "model": rng.choice(["qwen3", "qwen3_235b_tp8"]), "trees": 1, "nodes": _log(rng, 1, 128), "rows": rng.random() < 0.5}
    if kind == "accept":
        return {"kind": "accept", "trees": rng.randint(1, 8), "nodes": _log(rng, 2, 64), "layers": rng.randint(1, 8), "cap": rng.randint(128, 700)}
    return {"kind": "select", "model": "qwen3", "trees": _log(rng, 1, 32), "nodes": _log(rng, 2, 400)}


# ---- inputs -------------------------------------------------------------------------------------------------
def _gen(seed, purpose):
    return torch.Generator(device=DEV).manual_seed(seed * 1009 + purpose)


def _sizes(case):
    """Nodes of every tree: all alike for one tree, between three quarters and all of `nodes` in a batch."""
    n, B = case["nodes"], case.get("trees", 1)
    return [n if B == 1 or b == 0 or n < 4 else n - (b * 5) % (n // 4 + 1) for b in range(B)]


def _lens(case):
    """Context lengths: `ctx` for one sequence, between half and all of it in a batch."""
    L, B = case["ctx"], case.get("trees", 1)
    return [L if b == 0 else L - (b * 997) % (L // 2 + 1) for b in range(B)]


def _tree(n, rng, depth=6):
    """Parents of a draft tree: the root's first children, then children of random nodes that may still have some."""
    par, dep = [-1], [0]
    for i in range(1, n):
        p = 0 if i <= 4 else int(rng.integers(0, i))
        while dep[p] >= depth:
            p = par[p]
        par.append(p)
        dep.append(dep[p] + 1)
    return par, dep


def _trees(case, seed):
    rng = np.random.default_rng([seed, 7])
    sizes = _sizes(case)
    pairs = [_tree(n, rng) for n in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    T = int(off[-1])
    q = rng.uniform(0.05, 1.0, T).astype(np.float32)
    q[off[:-1]] = 1.0
    return SimpleNamespace(off=off, par=np.concatenate([p for p, _ in pairs]).astype(np.int32),
                           dep=np.concatenate([d for _, d in pairs]).astype(np.int64), q=q, T=T, B=len(sizes), sizes=sizes, rng=rng)


def _hidden(t, d, noise, dtype, seed):
    z = torch.randn(t.T, d, generator=_gen(seed, 11), device=DEV)
    x = z.clone()
    for b, n in enumerate(t.sizes):  # level by level
        lo = int(t.off[b])
        for level in range(1, int(t.dep[lo:lo + n].max()) + 1):
            rows = [lo + i for i in range(n) if t.dep[lo + i] == level]
            up = [lo + int(t.par[i]) for i in rows]
            x[rows] = x[up] + noise * z[rows]
    return x.to(dtype)


def _weights(c, seed, layer=0):
    g = _gen(seed, 100 + layer)
    dt = torch.bfloat16 if c.dtype == "bf16" else torch.float32

    def w(*shape):
        return torch.randn(*shape, generator=g, device=DEV, dtype=dt) * 0.02

    W = {"wq": w(c.Hq * c.D, c.d), "wk": w(c.Hkv * c.D, c.d), "wv": w(c.Hkv * c.D, c.d), "wo": w(c.d, c.Hq * c.D), "wg": w(c.E, c.d),
         "w_gate": w(c.E, c.F, c.d), "w_up": w(c.E, c.F, c.d), "w_down": w(c.E, c.d, c.F), "g_attn": 1 + 5 * w(c.d), "g_moe": 1 + 5 * w(c.d)}
    if c.n_shared:
        W.update(ws_gate=w(c.n_shared, c.F, c.d), ws_up=w(c.n_shared, c.F, c.d), ws_down=w(c.n_shared, c.d, c.F))
    return W


def _kv(c, B, cap, seed, layer=0):
    g = _gen(seed, 200 + layer)
    dt = torch.bfloat16 if c.dtype == "bf16" else torch.float32
    return (torch.randn(B, c.Hkv, cap, c.D, generator=g, device=DEV, dtype=dt),
            torch.randn(B, c.Hkv, cap, c.D, generator=g, device=DEV, dtype=dt))


def _head(c, seed):
    g = _gen(seed, 300)
    return (torch.randn(VOCAB, c.d, generator=g, device=DEV, dtype=torch.bfloat16) * 0.02,
            1 + 0.1 * torch.randn(c.d, generator=g, device=DEV, dtype=torch.bfloat16))


def _i32(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.int32), device=DEV)


def _zeros(*shape, dtype=torch.int32):
    return torch.zeros(*shape, dtype=dtype, device=DEV)


def _cost(kmax, c):
    k = np.arange(kmax + 1)
    return torch.as_tensor((1.0 + 0.05 * c.E * (1 - (1 - c.k / c.E) ** k)).astype(np.float32), device=DEV)


def _select_out(t):
    return SimpleNamespace(k_star=_zeros(t.B), keep=_zeros(t.T), par=_zeros(t.T), off=_zeros(t.B + 1), est=_zeros(t.B, dtype=torch.float32))


def _tokens(t, nxt, vocab):
    """Draft tokens: at most nodes one child carries the target's own token, so a path of a few nodes is accepted."""
    tok = t.rng.integers(0, vocab, t.T)
    for b, n in enumerate(t.sizes):
        lo = int(t.off[b])
        for i in range(1, n):
            if t.rng.random() < 0.4:
                tok[lo + i] = nxt[lo + t.par[lo + i]]
    return tok


def prepare(case, seed):
    s = SimpleNamespace(case=case, kind=case["kind"])
    t = s.t = _trees(case, seed)
    s.off, s.par, s.q = _i32(t.off), _i32(t.par), torch.as_tensor(t.q, device=DEV)
    if s.kind == "select":
        c = s.c = cfg_of(case)
        s.sel, s.cost, s.kmax = _select_out(t), _cost(max(t.sizes), c), max(t.sizes)
        s.x = _hidden(t, c.d, 0.5, torch.bfloat16, seed)
        s.rows = torch.zeros_like(s.x)
    elif s.kind == "accept":
        B, T, L = t.B, t.T, case["layers"]
        c = s.c = cfg_of({"model": "qwen3"}, d=256, E=16, k=2, F=32, Hq=4)  # (the context only lends its scratch to the acceptance)
        s.ctx = _Context(c, T, B, 16, 0)
        s.logits = 3 * torch.randn(T, VOCAB, generator=_gen(seed, 400), device=DEV)
        tok = t.rng.integers(0, VOCAB, T)
        rows = np.concatenate([t.off[b] + np.maximum(t.par[t.off[b]:t.off[b + 1]], 0) for b in range(B)])
        s.logits[torch.as_tensor(rows, device=DEV), torch.as_tensor(tok, device=DEV)] = torch.as_tensor(t.rng.uniform(13, 16, T).astype(np.float32), device=DEV)
        s.tok = _i32(tok)
        s.u_node = torch.as_tensor(t.rng.random(T).astype(np.float32), device=DEV)
        s.u_bonus = torch.as_tensor(t.rng.random(B).astype(np.float32), device=DEV)
        s.path, s.plen, s.bonus = _zeros(B, 16), _zeros(B), _zeros(B)
        kv = [_kv(c, B, case["cap"], seed, l) for l in range(L)]
        s.kc, s.vc = [k for k, _ in kv], [v for _, v in kv]
        g = _gen(seed, 500)
        s.kn, s.vn = ([torch.randn(T, c.Hkv, c.D, generator=g, device=DEV, dtype=torch.bfloat16) for _ in range(L)] for _ in range(2))
        s.len = _i32([case["cap"] - 20 - 7 * b for b in range(B)])
        s.len_out = _zeros(B)
    elif s.kind == "lm":
        c = s.c = cfg_of(case, E=16, k=2, F=32, Hq=4, Hkv=4)  # (layer shape unused: only the head is run)
        s.ctx = _Context(c, t.T, 1, 16, VOCAB)
        w, s.g_final = _head(c, seed)
        s.head = torch.empty_like(w).reshape(-1)
        ev.evict_pack_dense(ev.EVICT_BF16, w, VOCAB, c.d, s.head)
        s.x = _hidden(t, c.d, 0.5, torch.bfloat16, seed)
        s.next, s.best = _zeros(t.T), _zeros(t.T, dtype=torch.float32)
        s.tok = _i32(_tokens(t, t.rng.integers(0, VOCAB, t.T), VOCAB))
        s.path, s.plen, s.bonus = _zeros(1, 16), _zeros(1), _zeros(1)
        s.logits = _zeros(t.T, VOCAB, dtype=torch.float32) if case["rows"] else None
    else:
        c = s.c = cfg_of(case)
        dt = torch.bfloat16 if c.dtype == "bf16" else torch.float32
        lens = _lens(case)
        s.cap, s.len = max(lens), _i32(lens)
        s.x = _hidden(t, c.d, case["noise"], dt, seed)
        L = case.get("layers", 1)
        s.layers = []
        for l in range(L):
            s.layers.append(harness.DeviceLayer(c, _weights(c, seed, l), t.T, t.B, s.cap, DEV, VOCAB if s.kind == "iterate" else 0,
                                                s.layers[0].ctx if l else None))
        s.ctx = s.layers[0]
        kv = [_kv(c, t.B, s.cap, seed, l) for l in range(L)]
        s.out = torch.zeros_like(s.x)
        s.kn, s.vn = ([torch.zeros(t.T, c.Hkv, c.D, dtype=dt, device=DEV) for _ in range(L)] for _ in range(2))
        s.sel, s.cost, s.kmax = _select_out(t), _cost(max(t.sizes), c), max(t.sizes)
        nxt = t.rng.integers(0, VOCAB, t.T)
        s.next, s.tok = _i32(nxt), _i32(_tokens(t, nxt, VOCAB))
        s.path, s.plen, s.bonus = _zeros(t.B, 16), _zeros(t.B), _zeros(t.B)
        if s.kind == "iterate":
            w, s.g_final = _head(c, seed)
            s.head = torch.empty_like(w).reshape(-1)
            ev.evict_pack_dense(ev.EVICT_BF16, w, VOCAB, c.d, s.head)
            s.xin, s.logits = torch.zeros_like(s.x), _zeros(t.T, VOCAB, dtype=torch.float32)
            s.page = case["page"]
            s.table, paged = _to_pages(kv, s.page, t.rng)
            s.kc, s.vc = [k for k, _ in paged], [v for _, v in paged]
        else:
            s.kc, s.vc = [kv[0][0]], [kv[0][1]]
    torch.cuda.synchronize()
    return s


def _to_pages(kv, page, rng):
    """One sequence's caches cut into pages of `page` positions, the pages in random order."""
    _, H, cap, D = kv[0][0].shape
    n = -(-cap // page)
    at = rng.permutation(n)
    where = torch.as_tensor(at, device=DEV)
    out = []
    for pair in kv:
        pools = []
        for a in pair:
            full = torch.zeros(H, n * page, D, dtype=a.dtype, device=DEV)
            full[:, :cap] = a[0]
            pool = torch.zeros(n, H, page, D, dtype=a.dtype, device=DEV)
            pool[where] = full.view(H, n, page, D).transpose(0, 1)
            pools.append(pool)
        out.append(pools)
    return _i32(at).reshape(1, n), out


class _Context:
    """A library context that is destroyed with the state that holds it."""

    def __init__(self, c, tokens, batch, ctx, vocab):
        self.ctx = ev.evict_create(harness.model_desc(c, vocab), tokens, batch, ctx)

    def __del__(self):
        try:
            ev.evict_destroy(self.ctx)
        except Exception:
            pass


# ---- one pass -----------------------------------------------------------------------------------------------
def _select(s, ctx):
    o = s.sel
    ev.evict_select_prefix(ctx, s.off, s.par, s.q, s.t.B, s.t.T, s.cost, s.kmax, o.k_star, o.keep, o.par, o.off, o.est)


def run(s):
    t, c = s.t, s.c
    if s.kind == "select":
        o = s.sel
        _select(s, None)
        ev.evict_gather_rows(s.x, s.rows, c.d * 2, s.off, o.off, o.keep, t.B, t.T)
        return {"k_star": o.k_star, "keep": o.keep, "parent": o.par, "off": o.off, "est": o.est, "rows": s.rows}
    ctx = s.ctx.ctx
    if s.kind == "accept":
        ev.evict_accept_path_sampled(ctx, s.off, s.par, s.tok, s.logits, VOCAB, 0.8, s.u_node, s.u_bonus, t.B, t.T, s.path, 16, s.plen, s.bonus)
        ev.evict_kv_commit_stack(None, ev.EVICT_BF16, c.Hkv, c.D, s.kn, s.vn, s.off, s.path, 16, s.plen, s.kc, s.vc,
                                 s.kc[0].stride(0), s.kc[0].stride(1), s.len, s.case["cap"], s.len_out, t.B)
        return {"path": s.path, "len": s.plen, "bonus": s.bonus, "ctx": s.len_out, "k": s.kc, "v": s.vc}
    if s.kind == "lm":
        if s.case["rows"]:
            ev.evict_lm_head_logits(ctx, s.x, s.g_final, s.head, t.T, s.logits)
            return {"logits": s.logits}
        ev.evict_lm_head_argmax(ctx, s.x, s.g_final, s.head, t.T, s.next, s.best)
        ev.evict_accept_path(ctx, s.off, s.par, s.tok, s.next, 1, s.path, 16, s.plen, s.bonus)
        return {"next": s.next, "best": s.best, "path": s.path, "len": s.plen, "bonus": s.bonus}
    if s.kind == "iterate":
        o = s.sel
        _select(s, ctx)
        ev.evict_gather_rows(s.x, s.xin, c.d * 2, s.off, o.off, o.keep, 1, t.T)
        ev.evict_dynamic_tokens(ctx, o.off.data_ptr() + 4)
        n, H, page, D = s.kc[0].shape
        ev.evict_verify_stack_paged(ctx, [l.weights for l in s.layers], o.off, o.par, 1, t.T, s.kc, s.vc, H * page * D, page * D, s.table, n, page, n,
                                    s.len, s.cap, s.xin, s.out, s.kn, s.vn)
        ev.evict_lm_head_logits(ctx, s.out, s.g_final, s.head, t.T, s.logits)
        ev.evict_dynamic_tokens(ctx, None)
        return {"k_star": o.k_star, "keep": o.keep, "x": s.out, "logits": s.logits, "k": s.kn, "v": s.vn}
    step = s.case.get("step", False)
    if step:
        _select(s, ctx)
    ev.evict_verify_layer(ctx, s.layers[0].weights, s.off, s.par, t.B, t.T, s.kc[0], s.vc[0], s.kc[0].stride(0), s.kc[0].stride(1),
                          s.len, s.cap, s.x, s.out, s.kn[0], s.vn[0])
    got = {"x": s.out, "k": s.kn[0], "v": s.vn[0]}
    if step:
        ev.evict_accept_path(ctx, s.off, s.par, s.tok, s.next, t.B, s.path, 16, s.plen, s.bonus)
        got.update(k_star=s.sel.k_star, keep=s.sel.keep, path=s.path, len=s.plen, bonus=s.bonus)
    return got


# ---- what one pass cannot do without ------------------------------------------------------------------------
def _layer_work(c, sizes, lens, noise):
    eb = 2 if c.dtype == "bf16" else 4
    T = sum(sizes)
    alike = sum(n ** SPREAD[noise] for n in sizes)
    union = c.E * (1 - (1 - c.k / c.E) ** alike)
    dense = (c.Hq + 2 * c.Hkv) * c.D * c.d + c.Hq * c.D * c.d + c.E * c.d
    expert = 3 * c.d * c.F
    kv = 2 * c.Hkv * c.D * sum(lens)
    keys = sum(n * (L + 8) for n, L in zip(sizes, lens))
    return {"bytes": eb * (dense + (union + c.n_shared) * expert + kv + T * (2 * c.d + 2 * c.Hkv * c.D)),
            "flops": 2 * T * (dense + (c.k + c.n_shared) * expert) + 4 * keys * c.Hq * c.D}


def work(case):
    sizes = _sizes(case)
    T = sum(sizes)
    if case["kind"] == "select":
        return {"bytes": 24 * T + 2 * T * MODELS[case["model"]]["d"], "flops": 0}
    if case["kind"] == "accept":
        return {"bytes": 4 * T * VOCAB + 16 * case["layers"] * len(sizes) * 4 * 4 * 128, "flops": 3 * T * VOCAB}
    c = cfg_of(case)
    if case["kind"] == "lm":
        return {"bytes": 2 * c.d * (VOCAB + T) + (4 * T * VOCAB if case["rows"] else 0), "flops": 2 * T * c.d * VOCAB}
    if case["kind"] == "layer":
        return _layer_work(c, sizes, _lens(case), case["noise"])
    kept = max(1, int(0.35 * T))  # what the selection keeps of such a tree
    w = _layer_work(c, [kept], _lens(case), case["noise"])
    return {"bytes": case["layers"] * w["bytes"] + 2 * c.d * VOCAB + 4 * kept * VOCAB, "flops": case["layers"] * w["flops"] + 2 * kept * c.d * VOCAB}


def tolerance(case):
    if case["kind"] in ("select", "accept"):
        return "exact"  # copies, whole numbers and single 32-bit operations in a stated order
    if case["kind"] == "lm":
        return {"rel": 1e-4}
    if MODELS[case["model"]]["dtype"] == "f32":
        return {"rel": 1e-5}
    # One layer with its sums in another order: 1e-3 to 2e-3 measured, bf16 rounding at the hand-offs. Now and then a token whose
    # last expert is nearly tied goes to another one, which is about 4e-2 of that token's row; in a stack such a token stays
    # different in all layers that follow (1.6e-2 measured over four).
    if case["kind"] == "iterate":
        return {"rel": 3e-2}
    return {"rel": max(1e-2, min(3e-2, 4e-2 / math.sqrt(sum(_sizes(case)))))}


# ---- the same in 64 bits ------------------------------------------------------------------------------------
def _rms(x, gain, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _rotate(x, pos, theta):
    half = x.shape[-1] // 2
    a = pos[:, None] * theta ** (-torch.arange(half, device=DEV, dtype=torch.float64) / half)
    cos, sin = torch.cos(a)[:, None], torch.sin(a)[:, None]
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], -1)


def _layer64(c, W, off, par, dep, lens, K, V, x):
    T, G = x.shape[0], c.Hq // c.Hkv
    xn = _rms(x, W["g_attn"], c.eps)
    pos = torch.cat([L + torch.as_tensor(dep[off[b]:off[b + 1]], device=DEV).double() for b, L in enumerate(lens)])
    q = _rotate((xn @ W["wq"].double().T).view(T, c.Hq, c.D), pos, c.theta)
    k = _rotate((xn @ W["wk"].double().T).view(T, c.Hkv, c.D), pos, c.theta)
    v = (xn @ W["wv"].double().T).view(T, c.Hkv, c.D)
    o = torch.empty(T, c.Hq, c.D, dtype=torch.float64, device=DEV)
    for b, L in enumerate(lens):
        lo, hi = int(off[b]), int(off[b + 1])
        n = hi - lo
        see = torch.zeros(n, n, dtype=torch.bool)
        for i in range(n):
            p = i
            while p >= 0:
                see[i, p] = True
                p = int(par[lo + p])
        mask = torch.cat([torch.ones(n, L, dtype=torch.bool), see], 1).to(DEV)
        for g in range(c.Hkv):
            keys = torch.cat([K[b, g, :L].double(), k[lo:hi, g]])
            vals = torch.cat([V[b, g, :L].double(), v[lo:hi, g]])
            for h in range(g * G, (g + 1) * G):
                p = torch.softmax((q[lo:hi, h] @ keys.T / math.sqrt(c.D)).masked_fill(~mask, -math.inf), -1)
                o[lo:hi, h] = p @ vals
    h = x + o.reshape(T, -1) @ W["wo"].double().T
    hn = _rms(h, W["g_moe"], c.eps)
    score, idx = torch.topk(hn @ W["wg"].double().T, c.k, dim=-1)
    wts = torch.softmax(score, -1) if c.router_norm == "softmax" else torch.sigmoid(score) / torch.sigmoid(score).sum(-1, keepdim=True)
    out = h.clone()

    def mlp(rows, gate, up, down):
        return (torch.nn.functional.silu(rows @ gate.double().T) * (rows @ up.double().T)) @ down.double().T

    for e in range(c.E):
        tok, slot = torch.nonzero(idx == e, as_tuple=True)
        if len(tok):
            out.index_add_(0, tok, wts[tok, slot][:, None] * mlp(hn[tok], W["w_gate"][e], W["w_up"][e], W["w_down"][e]))
    for j in range(c.n_shared):
        out += mlp(hn, W["ws_gate"][j], W["ws_up"][j], W["ws_down"][j])
    return out, k, v


def _select64(t, c, kmax):
    """k* and the kept nodes of one tree."""
    score = [1.0]
    for i in range(1, t.T):
        score.append(float(np.float32(np.float32(score[t.par[i]]) * t.q[i])))
    order = sorted(range(t.T), key=lambda i: (-score[i], i))
    sums = np.cumsum([score[i] for i in order])[:kmax]
    cost = _cost(kmax, c).double().cpu().numpy()
    k_star = int(np.argmax(sums / cost[1:len(sums) + 1])) + 1
    return k_star, sorted(order[:k_star])


def exact(case, seed):
    t = _trees(case, seed)
    kind = case["kind"]
    if kind in ("select", "accept"):
        return None  # whole numbers and copies
    c = cfg_of(case)
    if kind == "lm":
        w, g_final = _head(c, seed)
        xn = _rms(_hidden(t, c.d, 0.5, torch.bfloat16, seed).double(), g_final, c.eps)
        logits = torch.cat([xn @ part.double().T for part in w.split(16384)], 1)
        if case["rows"]:
            return {"logits": logits}
        return {"next": None, "best": logits.max(-1).values, "path": None, "len": None, "bonus": None}
    dt = torch.bfloat16 if c.dtype == "bf16" else torch.float32
    lens = _lens(case)
    x = _hidden(t, c.d, case["noise"], dt, seed).double()
    if kind == "layer":
        K, V = _kv(c, t.B, max(lens), seed)
        x, k, v = _layer64(c, _weights(c, seed), t.off, t.par, t.dep, lens, K, V, x)
        got = {"x": x, "k": k, "v": v}
        if case.get("step", False):
            got.update(k_star=None, keep=None, path=None, len=None, bonus=None)
        return got
    n, keep = _select64(t, c, max(t.sizes))
    new = {v: i for i, v in enumerate(keep)}
    par = [new.get(int(t.par[v]), -1) for v in keep]
    x = x[keep]
    ks, vs = [], []

    def whole(a):  # the rows past the selected length are not written
        return torch.cat([a, torch.zeros(t.T - n, *a.shape[1:], dtype=a.dtype, device=DEV)])

    for l in range(case["layers"]):
        K, V = _kv(c, 1, lens[0], seed, l)
        x, k, v = _layer64(c, _weights(c, seed, l), [0, n], par, t.dep[keep], lens, K, V, x)
        ks.append(whole(k))
        vs.append(whole(v))
    w, g_final = _head(c, seed)
    xn = _rms(x, g_final, c.eps)
    return {"k_star": None, "keep": None, "x": whole(x), "logits": whole(torch.cat([xn @ part.double().T for part in w.split(16384)], 1)), "k": ks, "v": vs}
