"""Registers of the one-launch grouping as hipcc reports them (no GPU needed): its
round loop fills the register file, and what spills is written and read back
in every round."""
import os
import re
import subprocess

from paper_2306_01926_amd import build as gbuild


def test_grouping_kernels_hardly_spill():
    src = next(s for s in gbuild.SOURCES if s.endswith("ga_lloyd.hip"))
    cmd = [gbuild.hipcc(), *gbuild.DEVICE_FLAGS, "--cuda-device-only", "-c", src, "-o", os.devnull,
           "-Rpass-analysis=kernel-resource-usage"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    found = re.findall(r"Function Name: (\S*k_lloyd\S*?I\S*).*?VGPRs Spill: (\d+)", r.stderr, re.S)
    assert len(found) >= 4, found  # 1 to 4 blocks of 32 groups
    assert all(int(n) <= 2 for _, n in found), found
