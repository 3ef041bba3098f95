"""CPU checks of what the kernels' hand-written waits rest on, in the sources and in the gfx950 assembly of a build."""
import glob
import os
import re
import subprocess

import pytest

from paper_2510_12747_amd import build as lib_build


def test_every_wait_can_wait():
    """A count of 15 (lgkmcnt, four bits) or 63 (vmcnt, six bits) is the counter's largest value: no wait at all."""
    found = 0
    for path in sorted(glob.glob(os.path.join(lib_build.CSRC, "*"))):
        for m in re.finditer(r"(lgkmcnt|vmcnt)\((\d+)\)", open(path).read()):
            found += 1
            assert int(m[2]) < {"lgkmcnt": 15, "vmcnt": 63}[m[1]], (os.path.basename(path), m[0])
    assert found > 10


def loops(assembly):
    """{(function, header): instructions} of the loops that hold no other loop"""
    out, function, header, inner = {}, None, None, set()
    for line in assembly.splitlines():
        if m := re.match(r"(_Z\w+):", line):
            function, header = m[1], None
            continue
        if m := re.match(r"(?:\.L(BB\d+_\d+)|; %bb\.\d+):", line):
            block, of = m[1], re.search(r"Header=(BB\d+_\d+)", line)
            header = of[1] if of else None
        if "Loop Header" in line:                            # on the label's line, or under it after the parent's name
            header = block
        if "Inner Loop Header" in line:
            inner.add((function, header))
        if header and re.match(r"\t[a-z]", line):
            out.setdefault((function, header), []).append(line.split()[0])
    return {k: v for k, v in out.items() if k in inner}


@pytest.mark.parametrize("source", ["lcsa_attn_mfma.hip", "lcsa_attn_bwd_mfma.hip"])
def test_no_spilled_register_is_reloaded_in_a_loop_of_matrix_instructions(source, tmp_path):
    """The tile copies in flight share the vector-memory counter with a reload, and the compiler, which does not see them,
    waits for the reload with vmcnt(0): one reload per trip drains what the loop's own waits keep in flight."""
    out = tmp_path / "kernels.s"
    flags = [f for f in lib_build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.run(["/opt/rocm/bin/hipcc", *flags, "--offload-device-only", "-S", "-o", str(out), os.path.join(lib_build.CSRC, source)],
                   check=True, capture_output=True)
    found = {k: v for k, v in loops(out.read_text()).items() if any("mfma" in i for i in v)}
    assert len(found) >= 3, found.keys()
    for (function, header), instructions in found.items():
        assert not [i for i in instructions if i.startswith("scratch_load")], (function, header)
