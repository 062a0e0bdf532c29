"""TopK and the expert union behind it where the kernels change: one token per wavefront up to 16 tokens (27 with more than 128
experts) and from 33 on, a row of 16 lanes per token between, with 8 or 16 experts per lane and up to 16 picks; equal scores go to the
lower expert."""
import numpy as np
import pytest
import torch

import synth
from oracle import evict_oracle as orc

pytestmark = pytest.mark.gpu

pytest.importorskip("paper_2605_00342_amd")
import paper_2605_00342_amd as ev  # noqa: E402
from paper_2605_00342_amd import harness  # noqa: E402
from test_gpu_layer import run_case  # noqa: E402


@pytest.mark.parametrize("E,k", [(16, 1), (16, 16), (48, 3), (64, 8), (80, 8), (128, 16), (128, 17), (144, 8), (256, 16), (272, 4)])
@pytest.mark.parametrize("T", [1, 9, 16, 17, 19, 27, 28, 31, 32, 33, 65])
def test_topk_rule(E, k, T):
    cfg = synth.ModelCfg(f"topk{E}", "bf16", d=256, Hq=2, Hkv=1, D=64, E=E, k=k, F=32, theta=1e4,
                         router_norm="sigmoid" if E == 144 else "softmax")
    case = synth.make_case(cfg.name, n=T, L=20, seed=T + E, sigma=1.0, tree="random", cfg=cfg)
    wg = case["W"]["wg"]
    wg[E // 2:] = wg[: E - E // 2]  # every score twice, half the experts apart
    if T > 3:
        wg[3:7] = wg[3]             # and four neighbours alike
    got = run_case(case)
    s = np.asarray(got["router_logits"], np.float32)
    want = np.argsort(-s, axis=1, kind="stable")[:, :k]
    assert np.array_equal(got["topk_idx"], want)
    top = np.take_along_axis(s, want, 1).astype(np.float64)
    w = 1 / (1 + np.exp(-top)) if cfg.router_norm == "sigmoid" else np.exp(top - top[:, :1])
    np.testing.assert_allclose(got["topk_w"], w / w.sum(1, keepdims=True), rtol=0, atol=2e-6)  # (as test_gpu_layer.py)
    un = orc.expert_union(want, E)
    n = un["union_count"]
    assert got["union_count"] == n and np.array_equal(got["union_ids"][:n], un["union_ids"][:n])
    assert np.array_equal(got["hist"], un["hist"])


@pytest.mark.parametrize("E,k", [(64, 6), (256, 8)])
@pytest.mark.parametrize("bound,live", [(b, n) for b in (16, 17, 28, 32) for n in (1, 3, 16, 17, 27, 28, 32) if n <= b])
def test_counts_in_device_memory(E, k, bound, live):
    """A call that knows an upper bound of its nodes only: selection, weights and union are those of the live ones' scores."""
    cfg = synth.ModelCfg(f"topkdyn{E}", "bf16", d=256, Hq=2, Hkv=1, D=64, E=E, k=k, F=32, theta=1e4)
    case = synth.make_case(cfg.name, n=bound, L=20, seed=bound, sigma=1.0, tree="random", cfg=cfg)
    case["W"]["wg"][E // 2:] = case["W"]["wg"][: E // 2]  # every score twice
    layer = harness.DeviceLayer(cfg, case["W"], bound, 1, 20)
    dc = harness.DeviceCase(case)
    dc.tree_off = torch.tensor([0, live], dtype=torch.int32, device="cuda:0")
    ev.evict_dynamic_tokens(layer.ctx, dc.tree_off.data_ptr() + 4)
    dc.run(layer)
    got = dc.results()
    ev.evict_dynamic_tokens(layer.ctx, None)
    assert ev.evict_device_status(layer.ctx) == 0
    layer.close()
    s = np.asarray(got["router_logits"], np.float32)[:live]
    want = np.argsort(-s, axis=1, kind="stable")[:, :k]
    assert np.array_equal(got["topk_idx"][:live], want) and not got["topk_idx"][live:].any()
    top = np.take_along_axis(s, want, 1).astype(np.float64)
    w = np.exp(top - top[:, :1])
    np.testing.assert_allclose(got["topk_w"][:live], w / w.sum(1, keepdims=True), rtol=0, atol=2e-6)  # (as test_gpu_layer.py)
    un = orc.expert_union(want, E)
    n = un["union_count"]
    assert got["union_count"] == n and np.array_equal(got["union_ids"][:n], un["union_ids"][:n])
    assert np.array_equal(got["hist"], un["hist"])
