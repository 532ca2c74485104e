"""What the compiler says about the walk with draft distributions: its rows sit in registers, and a row that spills
goes to memory and back at every pass (24 sequences of V = 128256: 70 us with spills, 54 without)."""
import os
import re
import subprocess

from paper_2512_14069_amd import build


def test_no_kernel_of_the_walk_spills():
    src = os.path.join(build.CSRC, "radar_accept_q.hip")
    r = subprocess.run([build.HIPCC] + build.FLAGS + ["--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", src, "-o", os.devnull],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    scratch = [int(v) for v in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    spilled = [int(v) for v in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    assert len(names) == len(scratch) == len(spilled) and sum("accept_q_coop_kernel" in n for n in names) >= 8
    assert not any(scratch) and not any(spilled), [v for v in zip(names, scratch, spilled) if v[1] or v[2]]
