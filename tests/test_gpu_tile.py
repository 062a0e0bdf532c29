"""The tiled GEMM of the projections and the LM head at the sizes where its tiles end, and the expert kernels of few experts with
1, 15, 16, 17, ... tokens up to several slots (too few for the tiled ones, which test_gpu_tile_experts.py compares with these),
through the whole layer protocol (every stage against the CPU oracle)."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

ev = pytest.importorskip("paper_2605_00342_amd")
from paper_2605_00342_amd import harness  # noqa: E402
from test_gpu_layer import check_against_oracle, run_case  # noqa: E402

DEV = "cuda:0"


def layer_case(n, seed, d, F, E, k, n_shared=0, batch=1, Hq=8, Hkv=2, D=64, L=40, sigma=0.5):
    cfg = synth.ModelCfg(f"tile{d}_{F}", "bf16", d=d, Hq=Hq, Hkv=Hkv, D=D, E=E, k=k, F=F, n_shared=n_shared, theta=1e4)
    return synth.make_case(cfg.name, n=n, L=L, seed=seed, sigma=sigma, tree="random", batch=batch,
                           L_list=[L + 3 * b for b in range(batch)] if batch > 1 else None, cfg=cfg)


# every token goes to every expert (k = E): expert token counts are exactly n * batch
@pytest.mark.parametrize("n,batch", [(6, 1), (15, 1), (17, 1), (32, 1), (33, 1), (64, 1), (65, 1), (96, 1), (97, 1), (113, 1), (64, 3)])
def test_slot_edges(n, batch):
    case = layer_case(n, 300 + n, 2048, 768, 16, 16, batch=batch)
    check_against_oracle(case, run_case(case))


# the other contraction lengths of both projections; ragged expert sizes; strip groups with idle wavefronts; shared experts
@pytest.mark.parametrize("d,F,n_shared,n,k", [(2048, 1408, 1, 50, 4), (4096, 192, 0, 40, 4), (4096, 256, 1, 70, 4), (2048, 768, 2, 100, 2)])
def test_widths(d, F, n_shared, n, k):
    case = layer_case(n, 400 + n, d, F, 16, k, n_shared=n_shared)
    check_against_oracle(case, run_case(case))


# dense projections: token counts that pick each tile of strips x tokens in turn, with ragged last tiles (320 strips of 64
# blocks and 128 of 128 blocks; one rank's share: 80 strips of 128 and 256 of 32)
@pytest.mark.parametrize("n,batch", [(33, 1), (49, 1), (81, 1), (113, 1), (128, 1), (80, 2), (113, 2), (100, 3), (100, 4), (101, 6)])
def test_dense_tiles(n, batch):
    case = layer_case(n, 500 + n, 2048, 64, 16, 2, batch=batch, Hq=32, Hkv=4, D=128, L=20)
    check_against_oracle(case, run_case(case))


@pytest.mark.parametrize("n,batch", [(1, 1), (48, 1), (65, 1), (113, 1), (100, 3), (100, 5)])
def test_dense_tiles_of_a_share(n, batch):
    case = layer_case(n, 600 + n, 4096, 64, 16, 2, batch=batch, Hq=8, Hkv=1, D=128, L=20)
    check_against_oracle(case, run_case(case))


# LM head: score rows and arg max at every tile choice, ragged last tiles, strips that leave wavefronts idle; the count in
# device memory smaller than the bound
@pytest.mark.parametrize("d,T", [(2048, 33), (2048, 64), (2048, 65), (2048, 96), (2048, 97), (2048, 200), (4096, 9), (4096, 31),
                                 (4096, 50), (4096, 128)])
def test_lm_head_tiles(d, T):
    cfg = synth.ModelCfg("lm", "bf16", d=d, Hq=4, Hkv=4, D=64, E=16, k=2, F=32)
    V = 16672  # 1042 strips: enough for the tiled kernel at either length, no multiple of a workgroup's
    ctx = ev.evict_create(harness.model_desc(cfg, V), T, 1, 16)
    try:
        g = torch.Generator().manual_seed(d + T)
        x = torch.randn(T, d, generator=g).to(DEV, torch.bfloat16)
        w = (0.02 * torch.randn(V, d, generator=g)).to(DEV, torch.bfloat16)
        gain = (1 + 0.1 * torch.randn(d, generator=g)).to(DEV, torch.bfloat16)
        packed = torch.empty(V * d, dtype=torch.bfloat16, device=DEV)
        ev.evict_pack_dense(ev.EVICT_BF16, w, V, d, packed)
        xn = torch.zeros_like(x)
        logits = torch.full((T, V), -7.0, device=DEV)
        nxt, best = torch.zeros(T, dtype=torch.int32, device=DEV), torch.zeros(T, device=DEV)
        ev.evict_lm_head_logits(ctx, x, gain, packed, T, logits, xn)
        ev.evict_lm_head_argmax(ctx, x, gain, packed, T, nxt, best)
        want = xn.double() @ w.double().T
        # roundings of sums in eight chains add up like a random walk: 1.0e-7 (2048 columns) and 1.4e-7 (4096) of the rows'
        # root mean square measured, so 2e-6 is beyond 14 of its standard deviations (one chain: up to 4e-6 and 6e-6)
        assert float((logits - want).abs().max()) < 2e-6 * float(want.pow(2).mean().sqrt())
        val, idx = logits.max(-1)
        assert torch.equal(best, val) and torch.equal(nxt.long(), idx)
        few = torch.tensor([min(T, 18)], dtype=torch.int32, device=DEV)
        part = torch.full((T, V), -7.0, device=DEV)
        ev.evict_dynamic_tokens(ctx, few.data_ptr())
        ev.evict_lm_head_logits(ctx, x, gain, packed, T, part)
        ev.evict_dynamic_tokens(ctx, None)
        torch.cuda.synchronize()
        n = int(few.item())
        assert torch.equal(part[:n], logits[:n]) and bool((part[n:] == -7.0).all())
    finally:
        ev.evict_destroy(ctx)


# the tiled kernel adds up the same eight chains as the contraction split: the same score rows bit for bit up to 64 blocks;
# of 128 blocks the chains hold other blocks, as many of them, so the error against 64 bits is the same but for chance
@pytest.mark.parametrize("d,T", [(2048, 33), (2048, 64), (2048, 96), (2048, 128), (4096, 20), (4096, 64), (4096, 96), (4096, 128)])
def test_lm_head_sums(d, T):
    cfg = synth.ModelCfg("lm", "bf16", d=d, Hq=4, Hkv=4, D=64, E=16, k=2, F=32)
    V = 32000
    ctx = ev.evict_create(harness.model_desc(cfg, V), T, 1, 16)
    try:
        g = torch.Generator(device=DEV).manual_seed(d + T)
        x = torch.randn(T, d, generator=g, device=DEV).to(torch.bfloat16)
        w = (0.02 * torch.randn(V, d, generator=g, device=DEV)).to(torch.bfloat16)
        gain = (1 + 0.1 * torch.randn(d, generator=g, device=DEV)).to(torch.bfloat16)
        packed = torch.empty(V * d, dtype=torch.bfloat16, device=DEV)
        ev.evict_pack_dense(ev.EVICT_BF16, w, V, d, packed)
        xn, tiled, split = torch.zeros_like(x), torch.zeros(T, V, device=DEV), torch.zeros(T, V, device=DEV)
        ev.evict_lm_head_logits(ctx, x, gain, packed, T, tiled, xn)
        ev.evict_tune(ctx, "lm_nt", 2)
        ev.evict_lm_head_logits(ctx, x, gain, packed, T, split)
        torch.cuda.synchronize()
        if d == 2048:
            assert torch.equal(tiled, split)
        want = xn.double() @ w.double().T
        err = [float((a.double() - want).norm() / want.norm()) for a in (tiled, split)]
        assert err[0] < 1.05 * err[1], err  # (one chain of 64 / 128 blocks: 2.6 / 2.9 times)
    finally:
        ev.evict_destroy(ctx)


# the projections likewise, at the tiles of few and of many tokens (64 blocks: 512 QKV strips, 128 output strips)
@pytest.mark.parametrize("n,batch", [(33, 1), (65, 1), (100, 1), (113, 2), (100, 4)])
def test_dense_sums(n, batch):
    case = layer_case(n, 550 + n, 2048, 64, 16, 2, batch=batch, Hq=32, Hkv=16, D=64, L=20)
    tiled, split = run_case(case), run_case(case, tune={"dense_kernel": 0})
    for key in ("q", "k_new", "v_new", "h", "router_logits", "out"):
        assert np.array_equal(tiled[key], split[key]), key


# gate/up of 4096 columns: chunks cut by the slots on the device (about 35 slots of 16 pairs: four pairs each) or by the knob
def test_gateup_chunks():
    case = layer_case(40, 980, 4096, 256, 32, 4, n_shared=1)
    got = run_case(case)
    check_against_oracle(case, got)
    for chunk in (1, 2, 4):
        assert np.array_equal(got["out"], run_case(case, tune={"moe_chunk_gateup": chunk})["out"]), chunk


# many tokens: the router takes several expert strips per workgroup; short contractions have fewer slices than wavefronts
@pytest.mark.parametrize("d,E,n,batch", [(256, 128, 120, 5), (2048, 128, 120, 5), (512, 256, 100, 4), (96, 128, 128, 6)])
def test_router_strips(d, E, n, batch):
    case = layer_case(n, 900 + d, d, 32, E, 2, batch=batch, Hq=2, Hkv=2, D=64, L=5)
    check_against_oracle(case, run_case(case))


# ... whose scores are the same sums of slices then: no further from 64 bits than with one strip per workgroup (one, two and
# four slices per wavefront; one chain over two or four of them: 1.2 and 1.6 times as far)
def test_router_sums():
    err = []
    for batch in (1, 3, 8):
        case = layer_case(128, 950, 4096, 32, 256, 2, batch=batch, Hq=2, Hkv=2, L=5)
        got = run_case(case)
        want = np.asarray(got["h_norm"], np.float64) @ np.asarray(case["W"]["wg"], np.float64).T
        err.append(float(np.linalg.norm(got["router_logits"] - want) / np.linalg.norm(want)))
    assert max(err) < 1.05 * err[0], err


@pytest.mark.parametrize("vocab", [16, 65536, 65552, 131072, 131088])
@pytest.mark.parametrize("T", [1, 40])
def test_argmax_over_strips(vocab, T):
    """The arg max where its workgroup changes (4096 strips) and takes another trip (8192): every row of the head stands there twice,
    half the vocabulary apart, and the lower one is the answer; the greatest score sits in the first, the last and other strips."""
    d = 256
    cfg = synth.ModelCfg("lmargmax", "bf16", d=d, Hq=2, Hkv=1, D=64, E=16, k=2, F=64, theta=1e4)
    g = torch.Generator(device=DEV).manual_seed(vocab + T)
    w = (0.02 * torch.randn(vocab // 2, d, generator=g, device=DEV)).bfloat16()
    x = torch.randn(T, d, generator=g, device=DEV).bfloat16()
    where = torch.linspace(0, vocab // 2 - 1, T, device=DEV).long() if T > 1 else torch.tensor([vocab // 2 - 1], device=DEV)
    if vocab > T * 32:
        w[where] = x  # far above every other score
    w = torch.cat([w, w]).contiguous()
    ctx = ev.evict_create(harness.model_desc(cfg, vocab), T, 1, 16)
    head = torch.empty_like(w).reshape(-1)
    ev.evict_pack_dense(ev.EVICT_BF16, w, vocab, d, head)
    nxt, best = torch.zeros(T, dtype=torch.int32, device=DEV), torch.zeros(T, device=DEV)
    logits = torch.zeros(T, vocab, device=DEV)
    gain = torch.ones(d, dtype=torch.bfloat16, device=DEV)
    ev.evict_lm_head_argmax(ctx, x, gain, head, T, nxt, best)
    ev.evict_lm_head_logits(ctx, x, gain, head, T, logits)
    torch.cuda.synchronize()
    ev.evict_destroy(ctx)
    top = logits.max(dim=1).values
    assert torch.equal(best, top) and torch.equal(nxt.long(), (logits == top[:, None]).int().argmax(1))
    assert (nxt < vocab // 2).all() and (vocab <= T * 32 or torch.equal(nxt.long(), where))


@pytest.mark.parametrize("dtype,d", [("bf16", 256), ("bf16", 768), ("bf16", 1536), ("bf16", 3072), ("f32", 256), ("f32", 1024)])
@pytest.mark.parametrize("T", [1, 3, 16, 17, 40])
def test_score_rows_of_other_lengths(dtype, d, T):
    """Score rows by the contraction split (strips of 8 to 96 blocks, none of them 64 in bf16): products of the rows the head reports
    in 64 bits. An fp32 sum of d products is off by at most d * 2^-24 of the sum of their magnitudes."""
    V = 528
    cfg = synth.ModelCfg("lmrows", dtype, d=d, Hq=2, Hkv=1, D=64, E=16, k=2, F=64, theta=1e4)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device=DEV).manual_seed(d + T)
    w = (0.05 * torch.randn(V, d, generator=g, device=DEV)).to(td)
    x = torch.randn(T, d, generator=g, device=DEV).to(td)
    ctx = ev.evict_create(harness.model_desc(cfg, V), T, 1, 16)
    head = torch.empty_like(w).reshape(-1)
    ev.evict_pack_dense(ev.EVICT_BF16 if dtype == "bf16" else ev.EVICT_F32, w, V, d, head)
    rows, logits = torch.zeros_like(x), torch.full((T, V), float("nan"), device=DEV)
    ev.evict_lm_head_logits(ctx, x, torch.ones(d, dtype=td, device=DEV), head, T, logits, rows)
    torch.cuda.synchronize()
    ev.evict_destroy(ctx)
    got, rows, w = logits.double().cpu(), rows.double().cpu(), w.double().cpu()
    assert ((got - rows @ w.T).abs() <= d * 2.0 ** -24 * (rows.abs() @ w.abs().T)).all()
