"""The merge of the attention's partial softmaxes where its unrolling changes: up to 5, 9 and 17 splits in one go, a second batch of
17, the other held pairs up to 48 and batches of 16 beyond; with splits that are empty for the shorter sequence. In bf16 for the splits
of the 16-row attention kernel (chunks of 128 keys, one split more for the draft nodes) and of the 32-row one (chunks of 64)."""
import pytest

import synth

pytestmark = pytest.mark.gpu

pytest.importorskip("paper_2605_00342_amd")
from test_gpu_layer import check_against_oracle, run_case  # noqa: E402


@pytest.mark.parametrize("splits", [3, 5, 6, 9, 10, 17, 18, 34, 35, 48, 49, 60, 64, 65, 191, 192])
@pytest.mark.parametrize("D", [64, 128])
def test_f32_split_counts(splits, D):
    L = 64 * (splits - 2)  # 64 keys a split, two splits of draft nodes
    cfg = synth.ModelCfg("f32merge", "f32", d=128, Hq=2, Hkv=1, D=D, E=16, k=2, F=64, theta=1e4)
    case = synth.make_case(cfg.name, n=5, L=L, seed=splits, sigma=0.5, tree="random", batch=2, L_list=[L, 70], cfg=cfg)
    check_against_oracle(case, run_case(case))


@pytest.mark.parametrize("chunks", [4, 5, 8, 9, 16, 17, 31, 32])
@pytest.mark.parametrize("D", [64, 128])
def test_bf16_split_counts(chunks, D):
    # (experts of the usual width: 64 columns make a contribution of 50 roundings of the stored output, and half a rounding each
    # way, 1/100 to 6/100 of it seen, is what the protocol's bound of 5e-2 on the contribution is to tell from a wrong expert)
    cfg = synth.ModelCfg("bf16merge", "bf16", d=512, Hq=8, Hkv=2, D=D, E=32, k=4, F=192)
    case = synth.make_case(cfg.name, n=9, L=128 * chunks - 5, seed=chunks, sigma=0.5, tree="random", cfg=cfg)
    check_against_oracle(case, run_case(case))


@pytest.mark.parametrize("chunks", [4, 5, 8, 9, 16, 17, 31, 32])
def test_bf16_split_counts_of_128_keys(chunks):
    """128 columns on the 16-row kernel, which the knob keeps: the splits that 64 columns have above."""
    cfg = synth.ModelCfg("bf16merge", "bf16", d=512, Hq=8, Hkv=2, D=128, E=32, k=4, F=192)
    case = synth.make_case(cfg.name, n=9, L=128 * chunks - 5, seed=chunks, sigma=0.5, tree="random", cfg=cfg)
    check_against_oracle(case, run_case(case, tune={"attn_waves": 4}))


@pytest.mark.parametrize("splits", [1, 2, 5, 6, 9, 10, 17, 18, 31, 32])
def test_bf16_split_counts_of_64_keys(splits):
    cfg = synth.ModelCfg("bf16merge", "bf16", d=512, Hq=8, Hkv=2, D=128, E=32, k=4, F=192)
    case = synth.make_case(cfg.name, n=9, L=max(64 * (splits - 1) - 5, 0), seed=splits, sigma=0.5, tree="random", cfg=cfg)
    check_against_oracle(case, run_case(case))
