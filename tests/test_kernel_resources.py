"""CPU tier: the attention kernels keep their state in registers. The compiler's resource remarks
for gfx950, with the library's own flags, show no spilled vector register and no scratch memory in
any decode, prefill or fused kernel (a spill there is memory traffic inside the main loops)."""
import os
import re
import subprocess

import pytest

from paper_2607_23815_amd import build as b


@pytest.mark.parametrize("source", ["decode.hip", "prefill.hip", "mixed.hip"])
def test_no_spills_and_no_scratch(source, tmp_path):
    try:
        hipcc = b.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")
    r = subprocess.run([hipcc, "-O3"] + b.FLAGS +
                       ["--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(b.CSRC, source), "-o", str(tmp_path / "out.o")],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    spills = [int(n) for n in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    scratch = [int(n) for n in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    assert len(names) == len(spills) == len(scratch) >= 5, r.stderr[-2000:]
    bad = [x for x in zip(names, spills, scratch) if x[1] or x[2]]
    assert not bad, bad
