"""Publishing between workgroups, read from the generated gfx950 code: a flag
or a queue entry may only be stored once the write-back of the L2 before it has
finished, so every buffer_wbl2 needs an s_waitcnt vmcnt(0) before the next
access to memory.  (The compiler drops its own wait behind a write-back when
nothing else of the wave is outstanding; an entry was then seen before its
record, in one of a million instances, too seldom for a short run to show it.)
"""

import os
import re
import subprocess

import pytest

from paper_2103_00693_amd import build

SOURCES = [f for f in build.SOURCES if f.endswith(".hip")]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("isa")
    jobs = {}
    for f in SOURCES:
        dst = str(out / (f + ".asm"))
        cmd = [build.hipcc(), *build.COMMON, "--cuda-device-only", "-S", os.path.join(build.CSRC, f), "-o", dst]
        jobs[f] = (dst, subprocess.Popen(cmd, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL))
    text = {}
    for f, (dst, job) in jobs.items():
        assert job.wait() == 0, f
        text[f] = [re.sub(r"\s*;.*", "", line).strip() for line in open(dst)]
    return text


def _instructions(lines, at):
    return (line for line in lines[at:] if line and not line.startswith(".") and not line.endswith(":"))


def test_every_write_back_is_waited_for(assembly):
    found = 0
    for f, lines in assembly.items():
        for i, line in enumerate(lines):
            if not line.startswith("buffer_wbl2"):
                continue
            found += 1
            for nxt in _instructions(lines, i + 1):
                if re.match(r"s_waitcnt\b.*vmcnt\(0\)", nxt):
                    break
                assert not re.match(r"(global|flat|buffer|scratch|s_cbranch|s_branch|s_endpgm|s_barrier)", nxt), (f, i, nxt)
    assert found >= 5  # batch reduce for one and three words, batch solve in three word sizes
