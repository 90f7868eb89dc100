"""What the compiler reports of the kernels' registers (CPU only: the sources are compiled, nothing runs)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2606_06302_amd import build


@pytest.mark.parametrize("src", build.HIP_SOURCES)
def test_no_kernel_spills_to_scratch(src):
    """No kernel keeps registers in scratch memory: a reload is a load the compiler waits for with every load in
    flight, which drains the rings of loads that the attention kernels keep ahead of their products."""
    if not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)):
        pytest.skip("no HIP compiler")
    r = subprocess.run([build.HIPCC, *build.HIP_FLAGS, *build.HIP_EXTRA.get(src, []), "--cuda-device-only", "-S", "-o",
                        os.devnull, "-Rpass-analysis=kernel-resource-usage", os.path.join(build.CSRC, src)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    kernels = re.findall(r"Function Name: (\S+)", r.stdout)
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stdout)]
    assert kernels and len(kernels) == len(scratch)
    assert not any(scratch), [k for k, s in zip(kernels, scratch) if s]
