"""LM head of the contraction split: score rows and arg max on either side of the counts of tokens and strips where a workgroup keeps
them until its strips are done and where the strips are dealt out in one round, ragged last workgroups, candidates that tie across
workgroups, a count of tokens in device memory, both storage types."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

ev = pytest.importorskip("paper_2605_00342_amd")
from paper_2605_00342_amd import harness  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("dtype,d,V,Ts", [
    ("bf16", 2048, 16 * 4097, (1, 12, 13, 16, 17, 24, 25, 32)),   # one round from 13 tokens on: 17 strips each, the last one alone
    ("bf16", 2048, 16 * 4096, (13, 16, 17, 32)), ("bf16", 2048, 16 * 3, (1, 16, 17, 32)), ("bf16", 4096, 16 * 101, (1, 11)),
    ("bf16", 768, 16 * 3143, (1, 9, 16, 17, 33)), ("bf16", 1024, 16 * 2000, (1, 13, 17, 48)), ("bf16", 1536, 16 * 517, (2, 20)),
    ("f32", 256, 16 * 2001, (1, 14, 17, 40)),
    ("bf16", 2048, 16 * 2048, (1, 13, 32)), ("bf16", 2048, 16 * 2049, (1, 12, 16, 17, 32, 48)),  # kept by the workgroup from 2049 strips on,
    ("bf16", 768, 16 * 1536, (1, 16)), ("bf16", 768, 16 * 1537, (1, 16)), ("bf16", 4096, 16 * 2049, (1, 11, 13, 32)),  # of 24 blocks from 1537
])
def test_rows_and_best(dtype, d, V, Ts):
    cfg = synth.ModelCfg("lm", dtype, d=d, Hq=4, Hkv=4, D=64, E=16, k=2, F=64, theta=1e4)
    ctx = ev.evict_create(harness.model_desc(cfg, V), 64, 1, 16)
    try:
        dt = torch.bfloat16 if dtype == "bf16" else torch.float32
        gen = torch.Generator(device=DEV).manual_seed(d + V)
        w = (torch.randn(V, d, generator=gen, device=DEV) * 0.02).to(dt)
        w[V - 1] = w[V // 2]
        head = torch.empty_like(w).reshape(-1)
        ev.evict_pack_dense(harness.storage_code(dtype), w, V, d, head)
        gain = torch.ones(d, device=DEV, dtype=dt)
        x = torch.randn(64, d, generator=gen, device=DEV).to(dt)
        x[0] = w[V // 2] * 50  # the first token's best row is there twice
        for T in Ts:
            for live in sorted({T, max(1, T - 5)}):
                xn = torch.zeros(T, d, device=DEV, dtype=dt)
                rows = torch.full((T, V), -7.0, device=DEV)
                nxt = torch.full((T,), -7, dtype=torch.int32, device=DEV)
                best = torch.zeros(T, device=DEV)
                count = torch.tensor([live], dtype=torch.int32, device=DEV)
                if live < T:
                    ev.evict_dynamic_tokens(ctx, count)
                ev.evict_lm_head_logits(ctx, x, gain, head, T, rows, xn)
                ev.evict_lm_head_argmax(ctx, x, gain, head, T, nxt, best)
                ev.evict_dynamic_tokens(ctx, None)
                torch.cuda.synchronize()
                want = xn[:live].double() @ w.double().T
                err = (rows[:live].double() - want).norm() / want.norm()
                assert err < 1e-6, (T, live, float(err))  # fp32 sums of d products: a few 1e-7
                assert bool((rows[live:] == -7.0).all()) and bool((nxt[live:] == -7).all())
                assert torch.equal(best[:live], rows[:live].max(dim=1).values)  # the same sums
                low = torch.where(rows[:live] == best[:live, None], torch.arange(V, device=DEV)[None], V).min(dim=1).values
                assert torch.equal(nxt[:live].long(), low)
    finally:
        ev.evict_destroy(ctx)
