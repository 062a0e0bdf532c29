"""The tiled expert GEMM at sizes it is chosen for (at least 256 chunks): ragged experts from a single token to several slots,
shared experts, several pieces of work per workgroup, counts in device memory. Its sums are those of the strip kernels, so over
2048 columns every comparison is bit for bit; the strip kernels are checked against the CPU oracle elsewhere. The projections,
tiled or split, likewise."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

ev = pytest.importorskip("paper_2605_00342_amd")
from paper_2605_00342_amd import harness  # noqa: E402

DEV = "cuda:0"


def experts_case(d, F, E, k, n, batch, n_shared, Hq=8, Hkv=2, D=64):
    """A case whose experts are made on the device; score rows of unlike sizes, so that experts differ in tokens."""
    cfg = synth.ModelCfg("tile", "bf16", d=d, Hq=Hq, Hkv=Hkv, D=D, E=16, k=2, F=32, n_shared=n_shared, theta=1e4)
    case = synth.make_case(cfg.name, n=n, L=9, seed=d + F + n, sigma=0.5, tree="random", batch=batch,
                           L_list=[9 + 3 * b for b in range(batch)] if batch > 1 else None, cfg=cfg)
    g = torch.Generator(device=DEV).manual_seed(n)

    def w(*shape):
        return (0.02 * torch.randn(*shape, generator=g, device=DEV)).to(torch.bfloat16)

    W = dict(case["W"])
    W.update(w_gate=w(E, F, d), w_up=w(E, F, d), w_down=w(E, d, F))
    W["wg"] = (w(E, d) * torch.linspace(0.1, 2.0, E, device=DEV)[:, None]).to(torch.bfloat16)
    if n_shared:
        W.update(ws_gate=w(n_shared, F, d), ws_up=w(n_shared, F, d), ws_down=w(n_shared, d, F))
    return dict(case, cfg=replace(cfg, E=E, k=k, F=F), W=W)


class Runner:
    def __init__(self, case):
        self.case, self.T = case, int(case["tree_off"][-1])
        self.layer = harness.DeviceLayer(case["cfg"], case["W"], self.T, len(case["ctx_len"]), int(max(case["ctx_len"])))

    def __call__(self, tune, count=None):
        """One call; with `count` on the first nodes of a single tree, their number in device memory and T its bound."""
        ctx = ev.evict_create(self.layer.desc, self.T, len(self.case["ctx_len"]), int(max(self.case["ctx_len"])))
        old, self.layer.ctx = self.layer.ctx, ctx
        try:
            for key, value in tune.items():
                ev.evict_tune(ctx, key, value)
            dc = harness.DeviceCase(self.case)
            if count:
                dc.tree_off = harness.dev_i32([0, count])
                n = harness.dev_i32([count])
                ev.evict_dynamic_tokens(ctx, n.data_ptr())
            dc.run(self.layer)
            got = dc.results()
            ev.evict_dynamic_tokens(ctx, None)
            assert ev.evict_device_status(ctx) == 0
            return got
        finally:
            self.layer.ctx = old
            ev.evict_destroy(ctx)


STRIPS = {"moe_gateup_kernel": 1}  # (set, it asks for the strip kernels of both projections)


@pytest.mark.parametrize("d,F,E,k,n,batch,n_shared", [
    (2048, 768, 32, 8, 64, 1, 0), (2048, 768, 32, 8, 97, 1, 2), (2048, 768, 32, 8, 113, 3, 0), (2048, 768, 32, 8, 128, 7, 1),
    (2048, 1408, 32, 6, 90, 1, 1), (2048, 1408, 32, 6, 127, 4, 1),
])
def test_equals_strip_kernels(d, F, E, k, n, batch, n_shared):
    case = experts_case(d, F, E, k, n, batch, n_shared)
    run = Runner(case)
    got, strips, few = run({}), run(STRIPS), run({"moe_grid": 40})
    hist = got["hist"][got["hist"] > 0]
    assert len(set((hist + 15) // 16)) >= 3, hist  # several token tiles, not all alike
    for key in ("topk_idx", "out"):
        assert np.array_equal(got[key], strips[key]), key
        assert np.array_equal(got[key], few[key]), key + ", many pieces per workgroup"


# 4096 columns: the contraction split has the same chains but of other blocks, so up to one rounding of an activation to bf16
@pytest.mark.parametrize("F,E,k,n,batch,n_shared", [(192, 128, 8, 100, 2, 0), (192, 128, 8, 128, 5, 0), (256, 96, 8, 128, 1, 1)])
def test_long_contraction(F, E, k, n, batch, n_shared):
    run = Runner(experts_case(4096, F, E, k, n, batch, n_shared))
    got, split, few = run({}), run({"moe_gateup_kernel": 0}), run({"moe_grid": 40})
    assert np.array_equal(got["topk_idx"], split["topk_idx"]) and np.array_equal(got["out"], few["out"])
    rows = np.linalg.norm(got["out"] - split["out"], axis=1) / np.linalg.norm(split["out"], axis=1)
    assert rows.max() < 2.0 ** -8, rows.max()


# a bound of 128 with fewer nodes: every kernel is chosen by the bound
@pytest.mark.parametrize("count", [1, 16, 17, 70, 127])
def test_count_in_device_memory(count):
    run = Runner(experts_case(2048, 768, 32, 8, 128, 1, 1, Hq=16, Hkv=4, D=128))
    got, strips, split = run({}, count), run(STRIPS, count), run({"dense_kernel": 0}, count)
    for key in ("q", "k_new", "v_new", "h", "topk_idx", "out"):
        assert np.array_equal(got[key][:count], strips[key][:count]), key
        assert np.array_equal(got[key][:count], split[key][:count]), key
    for key in ("k_new", "v_new", "out"):
        assert not got[key][count:].any(), key + ": rows past the count are not written"
