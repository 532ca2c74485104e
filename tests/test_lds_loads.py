"""Loads that write LDS directly take their LDS address from m0, and the hardware wants one wait state between a scalar write of m0 and
such a load; inside assembly the compiler does not add it.  Read from the assembly of the sources as the library is built."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2512_14069_amd import build


def assembly(name):
    r = subprocess.run([build.HIPCC] + build.FLAGS + ["--offload-device-only", "-S", os.path.join(build.CSRC, name), "-o", "-"],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout


@pytest.fixture(scope="module")
def listings():
    names = [n for n in build.SOURCES if "load_lds" in open(os.path.join(build.CSRC, n)).read()]
    with ThreadPoolExecutor(4) as pool:
        return dict(zip(names, pool.map(assembly, names)))


def close_writes(text):
    """Loads into LDS whose predecessor in the program writes m0, and how many such loads there are."""
    found, loads, before = [], 0, ""
    for line in text.splitlines():
        line = line.split(";")[0].strip()
        if not line or line.endswith(":") or line.startswith("."):
            continue
        if re.match(r"(global|buffer|scratch)_load_lds|buffer_load_\S+ .*\blds\b", line):
            loads += 1
            if re.match(r"s_\S+ m0,", before):
                found.append((before, line))
        before = line
    return found, loads


def test_the_reading_finds_what_it_looks_for():
    text = "s_mov_b32 m0, s4\n;;#ASMEND\nglobal_load_lds_dwordx4 v1, s[2:3]\ns_mov_b32 m0, s5\ns_nop 0\nglobal_load_lds_dwordx4 v[1:2], off"
    assert close_writes(text) == ([("s_mov_b32 m0, s4", "global_load_lds_dwordx4 v1, s[2:3]")], 2)


def test_a_wait_state_between_m0_and_a_load_into_lds(listings):
    assert "radar_attention.hip" in listings
    for name, text in listings.items():
        found, loads = close_writes(text)
        assert loads > 0, name
        assert not found, (name, len(found), found[0])
