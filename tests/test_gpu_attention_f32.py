"""fp32 tree attention at the edges of its 64-key splits and 16-row tiles, both head dimensions, and on caches whose
strides are no multiple of a 16-byte piece, through the whole layer protocol (every stage against the CPU oracle)."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

pytest.importorskip("paper_2605_00342_amd")
from paper_2605_00342_amd import harness  # noqa: E402
from test_gpu_layer import check_against_oracle, run_case  # noqa: E402


def f32_case(n, Ls, D, Hq, Hkv, seed):
    cfg = synth.ModelCfg("f32attn", "f32", d=128, Hq=Hq, Hkv=Hkv, D=D, E=16, k=2, F=64, theta=1e4)
    return synth.make_case(cfg.name, n=n, L=Ls[0], seed=seed, sigma=0.5, tree="random", batch=len(Ls),
                           L_list=list(Ls) if len(Ls) > 1 else None, cfg=cfg)


@pytest.mark.parametrize("n,Ls,D,Hq,Hkv", [
    (1, [0], 64, 2, 2), (1, [63], 64, 4, 2), (8, [64], 64, 4, 2), (15, [65], 128, 1, 1), (16, [128], 64, 2, 2),
    (17, [1], 64, 1, 1), (63, [200], 128, 4, 1), (64, [129], 64, 8, 1), (65, [0], 64, 4, 2), (128, [70], 128, 8, 2),
    (20, [0, 64, 191], 64, 4, 2),
])
def test_edges(n, Ls, D, Hq, Hkv):
    case = f32_case(n, Ls, D, Hq, Hkv, 700 + n)
    check_against_oracle(case, run_case(case))


@pytest.mark.parametrize("pad", [1, 2, 3, 6])
def test_odd_strides(pad):
    """Heads and sequences any number of elements apart: the same results as densely packed caches, bit for bit."""
    case = f32_case(9, [70, 33], 64, 4, 2, 720)
    cfg = case["cfg"]
    layer = harness.DeviceLayer(cfg, case["W"], 18, 2, 70)
    want = harness.DeviceCase(case)
    want.run(layer)
    want = want.results()
    dc = harness.DeviceCase(case)
    head, seq = dc.head_stride + pad, cfg.Hkv * (dc.head_stride + pad) + pad
    for name in ("k_cache", "v_cache"):
        dense = getattr(dc, name)
        flat = torch.zeros(2 * seq, device=dense.device)
        flat.as_strided(dense.shape, (seq, head, cfg.D, 1)).copy_(dense)
        setattr(dc, name, flat)
    dc.head_stride, dc.seq_stride = head, seq
    dc.run(layer)
    got = dc.results()
    layer.close()
    for key in ("attn_out", "out", "k_new", "v_new"):
        assert (got[key] == want[key]).all(), key
