"""The tiled GEMM at the sizes where its tiles end, through the whole layer protocol (every stage against the CPU oracle):
experts with 1, 15, 16, 17, ... tokens up to several slots, strips that do not fill the last workgroup, shared experts."""
import pytest

import synth

pytestmark = pytest.mark.gpu

pytest.importorskip("paper_2605_00342_amd")
from test_gpu_layer import check_against_oracle, run_case  # noqa: E402


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
