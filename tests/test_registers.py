"""Registers of the kernels, read from the compiler's report on code compiled here, no GPU needed.  A vector register kept in
memory is worse than slow in the kernels that count their loads by hand: the compiler waits for every load in flight before it
takes the register back, the ones into LDS included, which undoes the distance at which the tiles are requested."""
import glob
import os
import re
import subprocess

import pytest

from paper_2312_17482_amd import build


def test_no_kernel_keeps_vector_registers_in_memory(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    jobs = [(f, subprocess.Popen([build.HIPCC] + build.FLAGS + [
        "-c", "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", f, "-o", str(tmp_path / (os.path.basename(f) + ".o"))],
        stdout=subprocess.DEVNULL, stderr=subprocess.PIPE, text=True)) for f in sorted(glob.glob(os.path.join(build.CSRC, "*.hip")))]
    kernels = 0
    for f, job in jobs:
        report = job.communicate(timeout=110)[1]
        assert job.returncode == 0, report
        names = re.findall(r"Function Name: (\S+)", report)
        spills = [int(x) for x in re.findall(r"VGPRs Spill: (\d+)", report)]
        scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", report)]
        assert len(names) == len(spills) == len(scratch)
        kernels += len(names)
        assert not any(spills) and not any(scratch), [k for k in zip(names, spills, scratch) if k[1] or k[2]]
    assert kernels > 50
