"""CPU checks of what the kernels' hand-written waits rest on."""
import glob
import os
import re

from paper_2510_12747_amd import build as lib_build


def test_every_wait_can_wait():
    """A count of 15 (lgkmcnt, four bits) or 63 (vmcnt, six bits) is the counter's largest value: no wait at all."""
    found = 0
    for path in sorted(glob.glob(os.path.join(lib_build.CSRC, "*"))):
        for m in re.finditer(r"(lgkmcnt|vmcnt)\((\d+)\)", open(path).read()):
            found += 1
            assert int(m[2]) < {"lgkmcnt": 15, "vmcnt": 63}[m[1]], (os.path.basename(path), m[0])
    assert found > 10
