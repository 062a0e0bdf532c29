"""GPU parity of acceptance under sampling (Sec. 2.1, Eq. 3) and of the full-score LM head.

Protocol: the oracle (float64, the paper's steps literally) runs on the scores the GPU side is
given, with the same random numbers. Accepted paths must be identical unless some tried child's
random number lies within 1e-5 of its acceptance threshold (such cases are skipped and counted).
The final draw is an inverse-CDF lookup decided in fp32 on the GPU, so the token is checked for
validity against the float64 cumulative distribution within 1e-5, and must carry mass."""
import numpy as np
import pytest
import torch

import synth
from oracle import evict_oracle as orc

pytestmark = pytest.mark.gpu

ev = pytest.importorskip("paper_2605_00342_amd")
from paper_2605_00342_amd import harness  # noqa: E402

DEV = "cuda:0"
MARGIN = 1e-5


def make_sampling_case(seed, sizes, V, spread=3.0, tree="bfs"):
    """Trees, peaked synthetic score rows and draft tokens taken (like a drafter's) from the most
    likely tokens under the parent's scores, so that acceptances and rejections both occur."""
    g = synth.philox(seed, 61)
    parents = []
    for n in sizes:
        parents.append(synth.tree_bfs_random(n, g) if tree == "bfs" else synth.tree_chain(n))
    tree_off, parent = synth.concat_trees(parents)
    T = int(tree_off[-1])
    logits = (spread * g.standard_normal((T, V))).astype(np.float32)
    tok = np.zeros(T, np.int32)
    for b, par in enumerate(parents):
        lo = int(tree_off[b])
        for u in range(len(par)):
            kids = [c for c in range(len(par)) if par[c] == u]
            top = np.argsort(-logits[lo + u])[: max(8, len(kids))]
            pick = g.permutation(top)[: len(kids)]
            for c, t in zip(kids, pick):
                tok[lo + c] = t
    u_node = (g.random(T) ** 3).astype(np.float32)  # skewed to small values: deeper accepted paths
    u_bonus = g.random(len(sizes)).astype(np.float32)
    return parents, tree_off, parent, logits, tok, u_node, u_bonus


def run_gpu(ctx, tree_off, parent, tok, logits, V, temp, u_node, u_bonus, stride):
    B, T = len(tree_off) - 1, int(tree_off[-1])
    i32 = torch.int32
    path = torch.full((B, stride), -7, dtype=i32, device=DEV)
    plen = torch.zeros(B, dtype=i32, device=DEV)
    bonus = torch.zeros(B, dtype=i32, device=DEV)
    lg = logits if isinstance(logits, torch.Tensor) else torch.from_numpy(logits).to(DEV)
    ev.evict_accept_path_sampled(ctx, harness.dev_i32(tree_off), harness.dev_i32(parent), harness.dev_i32(tok), lg, V,
                                 temp, torch.from_numpy(u_node).to(DEV), torch.from_numpy(u_bonus).to(DEV), B, T, path,
                                 stride, plen, bonus)
    torch.cuda.synchronize()
    return path.cpu().numpy(), plen.cpu().numpy(), bonus.cpu().numpy()


def check_against_oracle(parents, tree_off, logits, tok, u_node, u_bonus, temp, path, plen, bonus):
    """Returns the number of sequences skipped for a decision inside the margin."""
    skipped = 0
    P = orc.softmax_temperature(logits, temp)
    for b, par in enumerate(parents):
        lo, hi = int(tree_off[b]), int(tree_off[b + 1])
        rp, rb, trace, cdf = orc.accept_path_sampled(par, tok[lo:hi], P[lo:hi], u_node[lo:hi], u_bonus[b], with_trace=True)
        if any(abs(float(u_node[lo + c]) - p) < MARGIN for c, p, _ in trace):
            skipped += 1
            continue
        assert plen[b] == len(rp), f"sequence {b}: path length {plen[b]} vs {len(rp)}"
        assert list(path[b, : len(rp)]) == list(rp)
        assert np.all(path[b, len(rp):] == -1)
        t = int(bonus[b])
        below = cdf[t - 1] if t > 0 else 0.0
        assert cdf[t] - below > 0.0, f"sequence {b}: drawn token {t} has no mass left"
        assert below - MARGIN <= float(u_bonus[b]) <= cdf[t] + MARGIN, (b, t, below, float(u_bonus[b]), cdf[t])
    return skipped


@pytest.fixture(scope="module")
def ctx_small():
    cfg = synth.CONFIGS["tiny"]
    case = synth.make_case("tiny", n=8, L=64, seed=0)
    layer = harness.DeviceLayer(cfg, case["W"], max_tokens=512, max_batch=8, max_ctx=64)
    yield layer.ctx
    layer.close()


@pytest.mark.parametrize("seed,sizes,V,temp", [
    (1, [24], 1000, 1.0),
    (2, [40, 7, 64, 1], 1000, 0.7),
    (3, [128, 128], 5000, 1.3),
    (4, [33, 2, 90], 777, 0.5),       # vocabulary not a multiple of 64 or 16
    (5, [16] * 8, 50, 1.0),           # tiny vocabulary: repeated rejections drain most of the mass
])
def test_sampled_acceptance_matches_oracle(ctx_small, seed, sizes, V, temp):
    parents, tree_off, parent, logits, tok, u_node, u_bonus = make_sampling_case(seed, sizes, V)
    path, plen, bonus = run_gpu(ctx_small, tree_off, parent, tok, logits, V, temp, u_node, u_bonus, max(sizes))
    skipped = check_against_oracle(parents, tree_off, logits, tok, u_node, u_bonus, temp, path, plen, bonus)
    assert skipped <= 1
    assert plen.max() > 1 or len(sizes) == 1  # the cases do accept something


def test_full_vocabulary(ctx_small):
    V = 151936
    parents, tree_off, parent, logits, tok, u_node, u_bonus = make_sampling_case(11, [32], V, spread=4.0)
    path, plen, bonus = run_gpu(ctx_small, tree_off, parent, tok, logits, V, 0.8, u_node, u_bonus, 32)
    assert check_against_oracle(parents, tree_off, logits, tok, u_node, u_bonus, 0.8, path, plen, bonus) == 0


def test_low_temperature_is_the_greedy_rule(ctx_small):
    V = 400
    parents, tree_off, parent, logits, tok, u_node, u_bonus = make_sampling_case(21, [60, 60, 60], V, spread=5.0)
    nxt = logits.argmax(axis=1).astype(np.int32)
    # make some edges match the target's choice so that the greedy walk goes somewhere
    g = synth.philox(21, 62)
    for b, par in enumerate(parents):
        lo = int(tree_off[b])
        tok[lo:lo + len(par)] = synth.plant_draft_tokens(par, nxt[lo:lo + len(par)], V, g)
    path, plen, bonus = run_gpu(ctx_small, tree_off, parent, tok, logits, V, 0.01, u_node, u_bonus, 60)
    for b, par in enumerate(parents):
        lo, hi = int(tree_off[b]), int(tree_off[b + 1])
        rp, rb = orc.accept_path(par, tok[lo:hi], nxt[lo:hi])
        assert plen[b] == len(rp) and list(path[b, : len(rp)]) == list(rp) and bonus[b] == rb
    assert plen.max() > 1


def test_single_node_and_invalid_token(ctx_small):
    V = 300
    parents, tree_off, parent, logits, tok, u_node, u_bonus = make_sampling_case(31, [1, 5], V, tree="chain")
    tok[2] = V + 5  # the first draft node of the second tree carries an id outside the vocabulary
    u_node[:] = 0.0  # every valid child would be accepted
    path, plen, bonus = run_gpu(ctx_small, tree_off, parent, tok, logits, V, 1.0, u_node, u_bonus, 5)
    assert plen[0] == 1 and plen[1] == 1 and path[1, 0] == 0
    st = ev.evict_device_status(ctx_small)
    assert st != 0
    P = orc.softmax_temperature(logits, 1.0)
    for b, row in ((0, 0), (1, 1)):
        cdf = np.cumsum(P[row])
        t = int(bonus[b])
        assert (cdf[t - 1] if t else 0.0) - MARGIN <= float(u_bonus[b]) <= cdf[t] + MARGIN


def test_argument_errors(ctx_small):
    parents, tree_off, parent, logits, tok, u_node, u_bonus = make_sampling_case(1, [8], 64)
    with pytest.raises(ev.EvictError):
        run_gpu(ctx_small, tree_off, parent, tok, logits, 64, 0.0, u_node, u_bonus, 8)   # temperature 0
    with pytest.raises(ev.EvictError):
        run_gpu(None, tree_off, parent, tok, logits, 64, 1.0, u_node, u_bonus, 8)        # needs a context


def test_lm_head_logits_then_sampling():
    """Full-score LM head against the oracle's, then acceptance on those scores."""
    cfg = synth.CONFIGS["mini_bf16"]
    V, n = 2000, 48
    case = synth.make_case("mini_bf16", n=n, L=64, seed=9)
    g = synth.philox(9, 63)
    w_lm = synth.round_to_bf16((0.5 * g.standard_normal((V, cfg.d))).astype(np.float32))
    gain = synth.round_to_bf16((1.0 + 0.1 * g.standard_normal(cfg.d)).astype(np.float32))
    layer = harness.DeviceLayer(cfg, case["W"], max_tokens=n, max_batch=1, max_ctx=64, vocab=V)
    try:
        wlm_dev = harness.pack_lm_head(cfg, w_lm)
        x = harness.to_dev(case["x"], cfg.dtype)
        logits = torch.zeros(n, V, dtype=torch.float32, device=DEV)
        ev.evict_lm_head_logits(layer.ctx, x, harness.to_dev(gain, cfg.dtype), wlm_dev, n, logits)
        torch.cuda.synchronize()
        _, want = orc.lm_head_argmax(case["x"], gain, w_lm, cfg.eps, act="bf16")
        got = logits.cpu().numpy()
        assert np.linalg.norm(got - want) / np.linalg.norm(want) < 2e-2
        # acceptance on the GPU's own scores
        par = case["parent"]
        tok = np.zeros(n, np.int32)
        for u in range(n):
            kids = [c for c in range(n) if par[c] == u]
            top = np.argsort(-got[u])[: max(8, len(kids))]
            for c, t in zip(kids, g.permutation(top)):
                tok[c] = t
        u_node, u_bonus = g.random(n).astype(np.float32), g.random(1).astype(np.float32)
        tree_off = np.array([0, n], np.int32)
        path, plen, bonus = run_gpu(layer.ctx, tree_off, par, tok, logits, V, 1.0, u_node, u_bonus, n)
        assert check_against_oracle([par], tree_off, got, tok, u_node, u_bonus, 1.0, path, plen, bonus) == 0
    finally:
        layer.close()


@pytest.mark.parametrize("V", [1, 63, 64, 65, 1023, 1025, 16384 + 1, 32768, 65536 + 17, 200003])
def test_vocabulary_edges(ctx_small, V):
    """Row lengths around the batches, segments and pieces the kernels cut a score row into; some pieces and whole
    segments are empty, tokens near the ends are drawn."""
    kids = min(V, 8)
    sizes = [1, kids, 2 * kids]
    parents, tree_off, parent, logits, tok, u_node, u_bonus = make_sampling_case(100 + V % 97, sizes, V)
    for u in (0.0, 0.5, 1.0 - 2.0 ** -24):
        u_bonus[:] = u
        path, plen, bonus = run_gpu(ctx_small, tree_off, parent, tok, logits, V, 0.9, u_node, u_bonus, max(sizes))
        assert np.all((bonus >= 0) & (bonus < V))
        assert check_against_oracle(parents, tree_off, logits, tok, u_node, u_bonus, 0.9, path, plen, bonus) == 0


@pytest.mark.parametrize("V", [16384, 16385])
def test_short_and_long_rows_agree(ctx_small, V):
    """Either side of the row length from which the statistics are spread over several workgroups: every decision as the
    oracle's."""
    parents, tree_off, parent, logits, tok, u_node, u_bonus = make_sampling_case(41, [1, 9, 16, 30], V)
    path, plen, bonus = run_gpu(ctx_small, tree_off, parent, tok, logits, V, 0.8, u_node, u_bonus, 30)
    assert check_against_oracle(parents, tree_off, logits, tok, u_node, u_bonus, 0.8, path, plen, bonus) <= 1


@pytest.mark.parametrize("V", [49152, 49153, 65536, 65537, 151936, 16 * 64 * 150, 16 * 64 * 150 + 1, 16 * 64 * 152, 16 * 64 * 152 + 1])
@pytest.mark.parametrize("u", [0.0, 0.37, 1.0 - 2.0 ** -24])
def test_draw_rounds(ctx_small, V, u):
    """The longest rows of one workgroup, with pieces of 48 and 64, and the next; rows of one round and of one round more, of the pieces (150 elements)
    and of the segments (152 blocks of 64); the target at both ends of the cumulative sum: at 0 the first token that is not rejected
    takes it (every one has mass), just below 1 one of the last within the margin."""
    parents, tree_off, parent, logits, tok, u_node, _ = make_sampling_case(77, [5, 1], V, spread=2.0)
    logits[:, -200:] += 6.0  # (mass in the last segment and piece)
    path, plen, bonus = run_gpu(ctx_small, tree_off, parent, tok, logits, V, 0.9, u_node, np.full(2, u, np.float32), 8)
    assert check_against_oracle(parents, tree_off, logits, tok, u_node, np.full(2, u, np.float32), 0.9, path, plen, bonus) == 0
    if u == 0.0:
        for b, par in enumerate(parents):
            lo, last = int(tree_off[b]), path[b, plen[b] - 1]
            rejected = {int(tok[lo + c]) for c in range(len(par)) if par[c] == last}
            assert bonus[b] == min(set(range(len(par) + 1)) - rejected)


@pytest.mark.parametrize("V", [1000, 32000, 49153, 65537, 151936])
@pytest.mark.parametrize("empty", [(1,), (0, 2), (3,), (0, 1, 2, 3, 4, 5)])
def test_empty_trees_leave_their_neighbours_alone(ctx_small, V, empty):
    """Trees without nodes, between others (their offset is the next tree's root), at the end (past the last node) and in greater
    number than there are nodes: the other trees' paths and tokens are what they are without them, bit for bit, and an empty tree
    accepts its root alone."""
    parents, tree_off, parent, logits, tok, u_node, u_bonus = make_sampling_case(7, [2, 1] if len(empty) > 4 else [6, 9, 5], V)
    B, T = len(parents), int(tree_off[-1])
    want = run_gpu(ctx_small, tree_off, parent, tok, logits, V, 0.9, u_node, u_bonus, 16)
    assert check_against_oracle(parents, tree_off, logits, tok, u_node, u_bonus, 0.9, *want) == 0
    off, u, live = [0], [], []
    for b in range(B + 1):
        for _ in range(empty.count(b) if len(empty) <= 4 else 2):
            off.append(off[-1])
            u.append(0.999)
        if b < B:
            live.append(len(u))
            off.append(int(tree_off[b + 1]))
            u.append(u_bonus[b])
    assert off[-1] == T and (len(u) > T) == (len(empty) > 4)
    got = run_gpu(ctx_small, np.array(off, np.int32), parent, tok, logits, V, 0.9, u_node, np.array(u, np.float32), 16)
    for w, g in zip(want, got):
        assert np.array_equal(w, g[live])
    none = [b for b in range(len(u)) if b not in live]
    assert np.all(got[1][none] == 1) and np.all(got[0][none, 0] == 0) and np.all(got[0][none, 1:] == -1)
    assert np.all((got[2][none] >= 0) & (got[2][none] < V))


@pytest.mark.parametrize("V", [1000, 16385, 49153, 65537, 151936, 16 * 64 * 152 + 1])
def test_infinite_temperature_draws_every_token_alike(ctx_small, V):
    """A chain whose first two children are accepted (probability 1 / V, random number 0) and whose third is not: the bonus token is the one
    at u * (V - 1) among those left. Sums of ones are exact in fp32, so it is exactly that one."""
    g = synth.philox(V, 64)
    logits = (3.0 * g.standard_normal((4, V))).astype(np.float32)
    off, parent = np.array([0, 4], np.int32), np.array([-1, 0, 1, 2], np.int32)
    tok, u_node = np.array([0, 5, 6, 7], np.int32), np.array([0.0, 0.0, 0.0, 0.9], np.float32)
    for u in (0.0, 0.3, 0.5, 0.9):
        path, plen, bonus = run_gpu(ctx_small, off, parent, tok, logits, V, float("inf"), u_node, np.array([u], np.float32), 4)
        assert plen[0] == 3 and list(path[0]) == [0, 1, 2, -1]
        left = [t for t in range(V) if t != 7]
        assert bonus[0] == left[int(np.float32(u) * np.float32(V - 1))]


@pytest.mark.parametrize("V", [1000, 16385, 40000, 65537, 151936])
@pytest.mark.parametrize("low", [-np.inf, np.finfo(np.float32).min])
def test_masked_logits(ctx_small, V, low):
    """What a top-k or top-p filter leaves: rows with whole parts and segments (a sixteenth of the vocabulary each) without a token, tokens in
    one segment only, one single token, and an unmasked row beside them."""
    parents, tree_off, parent, logits, tok, u_node, u_bonus = make_sampling_case(51, [12, 1, 6, 1], V)
    T, seg = len(logits), -(-V // 16)
    keep = np.zeros((T, V), bool)
    for r in range(T):
        kind = r % 5
        if kind == 0: keep[r, :seg // 2] = keep[r, 9 * seg:9 * seg + 40] = True
        elif kind == 1: keep[r, 3 * seg + 1:5 * seg - 1] = True
        elif kind == 2: keep[r, V - 1] = True
        elif kind == 3: keep[r, np.argsort(-logits[r])[:50]] = True
        else: keep[r] = True
    keep[int(tree_off[3]), :] = False
    keep[int(tree_off[3]), 15 * seg:] = True  # (a tree of one node: the draw alone, from the last segment)
    for i in range(T):  # the draft tokens keep their place
        b = int(np.searchsorted(tree_off, i, side="right")) - 1
        if i > tree_off[b]: keep[int(tree_off[b]) + parent[i], tok[i]] = True
    logits[~keep] = low
    for u in (0.0, 0.4, 1.0 - 2.0 ** -24):
        u_bonus[:] = u
        path, plen, bonus = run_gpu(ctx_small, tree_off, parent, tok, logits, V, 0.9, u_node, u_bonus, 12)
        assert check_against_oracle(parents, tree_off, logits, tok, u_node, u_bonus, 0.9, path, plen, bonus) == 0
        for b in range(len(parents)):
            assert keep[int(tree_off[b]) + path[b, plen[b] - 1], bonus[b]]


@pytest.mark.parametrize("V", [1000, 65537])
def test_many_trees_and_statistics_of_an_earlier_call(V):
    """More than 64 trees, some of them empty, right after a call on the same context with other logits: the rows that a call leaves out (nodes
    without children, past 65536 logits) hold the earlier call's statistics, and none of them is used."""
    cfg = synth.CONFIGS["tiny"]
    sizes = [1 + (5 * b) % 4 for b in range(70)]
    parents, tree_off, parent, logits, tok, u_node, u_bonus = make_sampling_case(71, sizes, V)
    off, u, live = [0], [], []
    for b in range(70):
        if b % 9 == 4:
            off.append(off[-1])
            u.append(0.999)
        live.append(len(u))
        off.append(int(tree_off[b + 1]))
        u.append(u_bonus[b])
    off, u = np.array(off, np.int32), np.array(u, np.float32)
    ctx = ev.evict_create(harness.model_desc(cfg), int(tree_off[-1]), len(u), 16)
    try:
        run_gpu(ctx, off, np.where(parent > 0, 0, parent).astype(np.int32), tok, np.ascontiguousarray(-2.0 * logits[::-1]), V, 0.7, u_node, u, 4)
        path, plen, bonus = run_gpu(ctx, off, parent, tok, logits, V, 0.9, u_node, u, 4)
        assert check_against_oracle(parents, tree_off, logits, tok, u_node, u_bonus, 0.9, path[live], plen[live], bonus[live]) == 0
        assert plen.max() > 1 and ev.evict_device_status(ctx) == 0
    finally:
        ev.evict_destroy(ctx)


@pytest.mark.parametrize("V", [1000, 65537])
@pytest.mark.parametrize("bad", [[-1, 7], [-1, -3], [-1, 1], [-1, 7, 0, 5], [-1, 0, 2, 1]])
def test_invalid_parents_count_as_the_root(V, bad):
    """Every decision as with the root for a parent, right after a call with other logits; the status word says so. (The root's row is needed even
    where no node names it.)"""
    cfg = synth.CONFIGS["tiny"]
    n = len(bad)
    par = np.array([p if i == 0 or 0 <= p < i else 0 for i, p in enumerate(bad)], np.int32)
    g = synth.philox(V + n, 65)
    logits = (3.0 * g.standard_normal((n, V))).astype(np.float32)
    tok = np.array([0] + [int(np.argsort(-logits[par[i]])[i]) for i in range(1, n)], np.int32)
    off = np.array([0, n], np.int32)
    ctx = ev.evict_create(harness.model_desc(cfg), n, 1, 16)
    try:
        for u_node in (np.zeros(n, np.float32), np.full(n, 0.03, np.float32), np.full(n, 0.999, np.float32)):
            run_gpu(ctx, off, np.array(bad, np.int32), tok, np.ascontiguousarray(logits[::-1] * 1.5), V, 0.7, u_node, np.array([0.2], np.float32), 4)
            path, plen, bonus = run_gpu(ctx, off, np.array(bad, np.int32), tok, logits, V, 0.9, u_node, np.array([0.6], np.float32), 4)
            assert check_against_oracle([par], off, logits, tok, u_node, np.array([0.6], np.float32), 0.9, path, plen, bonus) == 0
        assert ev.evict_device_status(ctx) & ev.EVICT_ST_BAD_PARENT
    finally:
        ev.evict_destroy(ctx)
