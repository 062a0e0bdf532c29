"""Build-time check of the compiled kernels (no GPU): the production instances of the attention kernel must not
use scratch memory. A staging lambda that stops being inlined keeps its register arrays in scratch without any
spill being reported, and the kernel then runs at half its speed; the compiler's resource remarks show it."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")


@pytest.fixture(scope="module")
def resources(tmp_path_factory):
    """(scratch bytes, registers of both kinds) of every kernel of layer_kernels.hip, from the compiler's remarks."""
    from paper_2605_00342_amd import build as b
    src = os.path.join(b.CSRC, "layer_kernels.hip")
    obj = tmp_path_factory.mktemp("res") / "lk.o"
    cmd = [HIPCC, *b.FLAGS, "-Rpass-analysis=kernel-resource-usage", "-c", src, "-o", str(obj)]
    out = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, check=True).stdout
    name, seen, regs = None, {}, {}
    for line in out.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m and name:
            seen[name] = int(m.group(1))
        m = re.search(r"\b(?:VGPRs|AGPRs): (\d+)", line)
        if m and name:
            regs[name] = regs.get(name, 0) + int(m.group(1))
    return seen, regs


def test_attention_kernels_use_no_scratch(resources):
    seen, _ = resources
    attn = {k: v for k, v in seen.items() if "attn_partial_mfma_kernel" in k}
    assert len(attn) == 8, sorted(attn)  # head dimension 64 / 128 x 4 / 8 wavefronts x contiguous / paged
    assert all(v == 0 for v in attn.values()), attn
    router = {k: v for k, v in seen.items() if "router_logits_kernel" in k and "4BF16" in k}
    assert router and all(v <= 128 for v in router.values()), router


def test_fp32_attention_leaves_room_for_two_workgroups_per_cu(resources):
    """Four wavefronts per workgroup, one per SIMD: two workgroups share the 512 registers of a lane."""
    f32 = {k: v for k, v in resources[1].items() if "attn_partial_f32_kernel" in k}
    assert len(f32) == 2 and all(v <= 256 for v in f32.values()), f32


def test_tiled_gemm_spills_nothing(resources):
    tile = {k: v for k, v in resources[0].items() if "gemm_tile_kernel" in k}
    assert tile and all(v == 0 for v in tile.values()), tile
