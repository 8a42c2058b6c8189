"""What the compiler makes of the kernels that hold their working set in registers: none of it may lie in scratch
memory (an array that is not promoted to registers counts as no spill, but every access to it goes to memory)."""
import os
import re
import subprocess

import pytest

from paper_2511_01884_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _scratch(source):
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    cmd = [HIPCC, *flags, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
           os.path.join(build.CSRC, source), "-o", os.devnull]
    out = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert out.returncode == 0, out.stdout
    names = re.findall(r"Function Name: (\S+)", out.stdout)
    sizes = [int(n) for n in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", out.stdout)]
    assert names and len(names) == len(sizes)
    return dict(zip(names, sizes))


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no compiler")
@pytest.mark.parametrize("source", ["ff_rowmean.hip", "ff_xent.hip", "ff_split.hip"])
def test_no_scratch_memory(source):
    used = {name: size for name, size in _scratch(source).items() if size}
    assert not used, used
