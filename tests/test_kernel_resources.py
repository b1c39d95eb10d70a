"""What the compiler reports of the kernels' registers (compiled here for
gfx950, no GPU needed): none spills a vector register or uses scratch memory.
A reload in a tile loop waits for every copy in flight."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2310_08152_amd import build

SOURCES = ("compact", "decode", "meta", "prefill")


@pytest.mark.parametrize("source", SOURCES)
def test_no_kernel_spills(source, tmp_path):
    if not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")):
        pytest.skip("no hipcc")
    r = subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, "-Rpass-analysis=kernel-resource-usage",
                        "--cuda-device-only", "-c", os.path.join(build.CSRC, source + ".hip"),
                        "-o", str(tmp_path / "k.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    spilled = [int(x) for x in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    assert names and len(names) == len(scratch) == len(spilled)
    assert not [n for n, s, v in zip(names, scratch, spilled) if s or v]
