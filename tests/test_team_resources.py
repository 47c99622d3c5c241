"""Registers of the kernels that are compiled for a number of waves per SIMD (no GPU
needed): the teams of the direct sum (FP32 four waves, so 128 registers; FP64 two)
and the Barnes-Hut leaf pairs (four).  None may spill: their hot loops use nearly all
registers, and a change nearby can push them over."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2106_12655_amd import build

HIPCC = build._hipcc()


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC),
                    reason="hipcc not available")
def test_teams_and_leaf_pairs_fit_their_waves(tmp_path):
    out = str(tmp_path / "lk_ds.s")
    r = subprocess.run([HIPCC, *build.HIPFLAGS, "--cuda-device-only", "-S",
                        os.path.join(build.CSRC, "lk_ds.hip"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    found = re.findall(r"\.agpr_count:\s+(\d+).*?\.name:\s+(\S+).*?"
                       r"\.vgpr_count:\s+(\d+).*?\.vgpr_spill_count:\s+(\d+)",
                       open(out).read(), re.S)
    teams = [f for f in found if "ds_team" in f[1]]
    near = [f for f in found if "bh_near_k" in f[1]]
    assert len(teams) == 6 and len(near) == 2
    for agpr, name, vgpr, spill in teams + near:
        fp64 = re.search(r"ds_teamI[fd]d", name) is not None
        assert int(vgpr) + int(agpr) <= (256 if fp64 else 128), (name, vgpr, agpr)
        assert int(spill) == 0, (name, spill)
