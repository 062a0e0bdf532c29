"""bf16 tree attention with several whole chunks, ragged chunks and draft nodes per workgroup: row counts around the tile and
workgroup edges, empty contexts, batches, both head dimensions; and the paged form bit for bit against the contiguous one.
(The launch-shape knob lowers the call size from which 8-wavefront workgroups are chosen.)"""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

ev = pytest.importorskip("paper_2605_00342_amd")
from paper_2605_00342_amd import harness  # noqa: E402
from test_gpu_layer import check_against_oracle, run_case  # noqa: E402
import test_gpu_paged as paged  # noqa: E402


@pytest.mark.parametrize("n,Ls,D,G,wgs", [
    (31, [130], 128, 8, 2), (32, [128], 128, 8, 2), (33, [300], 128, 8, 2), (65, [257], 64, 8, 2), (128, [700], 128, 8, 16),
    (128, [129], 64, 2, 2), (100, [384], 64, 4, 2), (64, [0, 1, 200], 128, 4, 2), (47, [513, 127], 128, 8, 8),
])
def test_edges(n, Ls, D, G, wgs):
    cfg = synth.ModelCfg("wide", "bf16", d=256, Hq=2 * G, Hkv=2, D=D, E=16, k=2, F=64, theta=1e4)
    case = synth.make_case(cfg.name, n=n, L=Ls[0], seed=800 + n, sigma=0.5, tree="random", batch=len(Ls),
                           L_list=list(Ls) if len(Ls) > 1 else None, cfg=cfg)
    check_against_oracle(case, run_case(case, tune={"attn_target_wgs": wgs}))


@pytest.mark.parametrize("cfg_name,Ls,P", [("mini_bf16", [300], 16), ("mini_bf16", [129, 500], 64), ("mini_sigmoid", [260], 32)])
def test_paged_equals_contiguous(cfg_name, Ls, P):
    case, cfg, Ws, Ks, Vs, pools, table, n_pages = paged.build(cfg_name, 128, Ls, P, 90, 0)
    dev = paged.Dev(case, cfg, Ws, Ks, Vs, pools, table, n_pages, P, max(Ls))
    try:
        ev.evict_tune(dev.ctx, "attn_target_wgs", 2)
        ctx_len = harness.dev_i32(case["ctx_len"])
        a = dev.run_contiguous(case["tree_off"], case["parent"], ctx_len, max(Ls), case["x"])
        b = dev.run_paged(case["tree_off"], case["parent"], ctx_len, max(Ls), case["x"])
        torch.cuda.synchronize()
        assert torch.equal(a[0], b[0]) and all(torch.equal(x, y) for x, y in zip(a[1] + a[2], b[1] + b[2]))
    finally:
        dev.close()
