"""No kernel keeps registers in scratch memory.  A 64-bit address of which the compiler had put one half into an accumulation register and
the other into scratch was reloaded without the first (backward, float, d > 128): the kernel read beyond all memory."""
import concurrent.futures
import os
import re
import subprocess

from paper_2510_12747_amd import build


def test_no_kernel_spills_registers(tmp_path):
    def assembly(source):
        out = tmp_path / (source + ".s")
        flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared", "-Wall")]
        subprocess.run(["/opt/rocm/bin/hipcc", *flags, "-w", "-S", "--cuda-device-only", "-o", str(out), os.path.join(build.CSRC, source)],
                       check=True, capture_output=True)
        return out.read_text()

    with concurrent.futures.ThreadPoolExecutor(4) as pool:
        texts = list(pool.map(assembly, build.SOURCES))
    kernels = 0
    for source, text in zip(build.SOURCES, texts):
        for name, scratch, spilled in re.findall(r"\.name: +(\S+)\n\s+\.private_segment_fixed_size: (\d+).*?\.vgpr_spill_count: (\d+)", text, re.S):
            kernels += 1
            assert int(scratch) == 0 and int(spilled) == 0, (source, name, scratch, spilled)
    assert kernels > 60
