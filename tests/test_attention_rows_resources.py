"""Build-time check (no GPU): the attention kernel of 32 rows per wavefront keeps its state in registers, none in scratch memory, and few
enough of both registers and LDS for two workgroups of four wavefronts per CU."""
import os
import re
import subprocess

import pytest

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")


def test_two_workgroups_per_cu(tmp_path):
    from paper_2605_00342_amd import build as b
    cmd = [HIPCC, *b.FLAGS, "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(b.CSRC, "attn_rows.hip"), "-o", str(tmp_path / "a.o")]
    out = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, check=True).stdout

    def numbers(what):
        return [int(x) for x in re.findall(re.escape(what) + r": (\d+)", out)]

    vgprs, agprs = numbers(" VGPRs"), numbers(" AGPRs")
    assert len(vgprs) == 3 and all(v + a <= 256 for v, a in zip(vgprs, agprs)), (vgprs, agprs)  # contiguous, pages, small pages
    assert numbers("ScratchSize [bytes/lane]") == [0, 0, 0]
    assert all(l <= 80 * 1024 for l in numbers("LDS Size [bytes/block]"))
