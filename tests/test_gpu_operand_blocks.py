"""Token operands kept in blocks of 16 tokens, of 1, 2, 4 or 8 in calls of up to 8: counts around whole blocks, and the final norm's
rows that a caller asks for, at any address."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

ev = pytest.importorskip("paper_2605_00342_amd")
from paper_2605_00342_amd import harness  # noqa: E402
from test_gpu_layer import check_against_oracle, run_case  # noqa: E402

DEV = "cuda:0"


CONFIGS = {"mini_bf16": synth.CONFIGS["mini_bf16"], "tiny": synth.CONFIGS["tiny"],  # heads of 128 and of 64 columns
           "bf16_64": synth.ModelCfg("bf16_64", "bf16", d=512, Hq=8, Hkv=2, D=64, E=32, k=4, F=192),
           "f32_128": synth.ModelCfg("f32_128", "f32", d=256, Hq=4, Hkv=2, D=128, E=16, k=2, F=128, theta=1e4)}


@pytest.mark.parametrize("config", list(CONFIGS))
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 33, 49, 113])
def test_layer_token_counts(config, n):
    case = synth.make_case(config, n=n, L=90, seed=n, sigma=0.5, tree="random", cfg=CONFIGS[config])
    for tune in ({}, {"dense_kernel": 1}):  # (contraction split and strip per wavefront)
        check_against_oracle(case, run_case(case, tune=tune))


@pytest.mark.parametrize("T", [1, 2, 3, 6, 9, 16, 17, 40])
@pytest.mark.parametrize("shift", [0, 1, 4])
def test_rows_of_the_final_norm(T, shift):
    """x_norm_out, `shift` elements past a 16-byte boundary, holds the rows that the scores were formed from."""
    d, V = 256, 1024
    cfg = synth.ModelCfg("lmrows", "bf16", d=d, Hq=2, Hkv=1, D=64, E=16, k=2, F=64, theta=1e4)
    g = torch.Generator().manual_seed(T)
    x = torch.randn(T, d, generator=g).bfloat16()
    gain = (1 + 0.1 * torch.randn(d, generator=g)).bfloat16()
    w = (0.05 * torch.randn(V, d, generator=g)).bfloat16()
    ctx = ev.evict_create(harness.model_desc(cfg, V), T, 1, 16)
    head = harness.pack_lm_head(cfg, w.float().numpy())
    logits = torch.zeros(T, V, device=DEV)
    buf = torch.full((T * d + 32,), 7.0, dtype=torch.bfloat16, device=DEV)
    ev.evict_lm_head_logits(ctx, x.to(DEV), gain.to(DEV), head, T, logits, buf[shift:])
    torch.cuda.synchronize()
    ev.evict_destroy(ctx)
    rows = buf[shift:shift + T * d].view(T, d).float().cpu()
    xf = x.double()
    want = xf / torch.sqrt((xf * xf).mean(-1, keepdim=True) + cfg.eps) * gain.double()
    np.testing.assert_allclose(rows.numpy(), want.numpy(), rtol=2 ** -8 * 1.01, atol=0)  # one bf16 rounding
    assert (buf[:shift] == 7.0).all() and (buf[shift + T * d:] == 7.0).all()
    # 256 products of rounded values in fp32 sums: 256 * 2^-24 of the sum of magnitudes
    got, ref = logits.double().cpu(), rows.double() @ w.double().T
    assert ((got - ref).abs() <= 256 * 2.0 ** -24 * (rows.double().abs() @ w.double().abs().T)).all()


@pytest.mark.parametrize("dtype,d,bound", [("bf16", 512, 8), ("bf16", 512, 16), ("bf16", 512, 40), ("f32", 256, 32), ("bf16", 2048, 64)])
@pytest.mark.parametrize("live", [1, 2, 3, 5, 8, 9, 64])
def test_head_of_a_count_in_device_memory(dtype, d, bound, live):
    """A head that knows an upper bound of its tokens only (and has the operand blocks of that bound) gives the rows of the live ones,
    their scores and arg max as the products of the rows in 64 bits (d * 2^-24 of the sum of magnitudes) and touches no others; a
    count above the bound is the bound."""
    V, n = 32768, min(live, bound)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    cfg = synth.ModelCfg("lmcount", dtype, d=d, Hq=2, Hkv=1, D=64, E=16, k=2, F=64, theta=1e4)
    g = torch.Generator(device=DEV).manual_seed(bound + live)
    x = torch.randn(bound, d, generator=g, device=DEV).to(td)
    w = (0.05 * torch.randn(V, d, generator=g, device=DEV)).to(td)
    ctx = ev.evict_create(harness.model_desc(cfg, V), bound, 1, 16)
    head = torch.empty_like(w).reshape(-1)
    ev.evict_pack_dense(ev.EVICT_BF16 if dtype == "bf16" else ev.EVICT_F32, w, V, d, head)
    gain, count = torch.ones(d, dtype=td, device=DEV), torch.tensor([live], dtype=torch.int32, device=DEV)
    rows, logits = torch.zeros_like(x), torch.full((bound, V), -7.0, device=DEV)
    nxt, best = torch.full((bound,), -1, dtype=torch.int32, device=DEV), torch.zeros(bound, device=DEV)
    ev.evict_dynamic_tokens(ctx, count.data_ptr())
    ev.evict_lm_head_logits(ctx, x, gain, head, bound, logits, rows)
    ev.evict_lm_head_argmax(ctx, x, gain, head, bound, nxt, best)
    ev.evict_dynamic_tokens(ctx, None)
    torch.cuda.synchronize()
    ev.evict_destroy(ctx)
    ref, mag = rows[:n].double() @ w.double().T, rows[:n].double().abs() @ w.double().abs().T
    assert ((logits[:n].double() - ref).abs() <= d * 2.0 ** -24 * mag).all() and bool((logits[n:] == -7.0).all())
    val, idx = logits[:n].max(-1)
    assert torch.equal(best[:n], val) and torch.equal(nxt[:n].long(), idx)
    assert not rows[n:].any() and bool((nxt[n:] == -1).all())


@pytest.mark.parametrize("T,d", [(1, 256), (9, 256), (40, 256), (700, 2048)])
@pytest.mark.parametrize("over", ["x", "x+1", "x-1", "x+8", "gain"])
def test_rows_of_the_final_norm_over_its_inputs(T, d, over):
    """x_norm_out over the rows (the same, one or eight further on, one before) or the gain that the norm reads: what it is and
    what the scores are elsewhere."""
    V = 1024
    cfg = synth.ModelCfg("lmover", "bf16", d=d, Hq=2, Hkv=1, D=64, E=16, k=2, F=64, theta=1e4)
    g = torch.Generator(device=DEV).manual_seed(T)
    x = torch.randn(T, d, generator=g, device=DEV).bfloat16()
    gain = (1 + 0.1 * torch.randn(d, generator=g, device=DEV)).bfloat16()
    ctx = ev.evict_create(harness.model_desc(cfg, V), T, 1, 16)
    head = harness.pack_lm_head(cfg, (0.05 * np.random.default_rng(T).standard_normal((V, d))).astype(np.float32))
    want_rows, want, got = torch.zeros_like(x), torch.zeros(T, V, device=DEV), torch.zeros(T, V, device=DEV)
    ev.evict_lm_head_logits(ctx, x, gain, head, T, want, want_rows)
    buf = torch.zeros((T + 16) * d, dtype=torch.bfloat16, device=DEV)
    at = 8 * d
    xin = buf[at:at + T * d].view(T, d)
    xin.copy_(x)
    if over == "gain":
        gain = buf[at + T * d - d // 2:at + T * d + d - d // 2].copy_(gain)  # (half under the rows, half behind)
        xin, out = x, buf[at:]
    else:
        out = buf[at + d * int(over[1:] or 0):]
    ev.evict_lm_head_logits(ctx, xin, gain, head, T, got, out)
    torch.cuda.synchronize()
    ev.evict_destroy(ctx)
    assert torch.equal(out[:T * d].view(T, d), want_rows) and torch.equal(got, want)
