"""Rings of LDS stages that other wavefronts' direct-to-LDS loads refill behind a barrier: the wait before that barrier must cover this wavefront's
reads of the stage (lgkmcnt), not only the loads that have to have landed (vmcnt).  Matrix instructions have no side effects, so nothing else holds
them, and the compiler's own wait for their operands, in front of the barrier.  Read off the sources: such a race cannot be shown by running it."""
import os
import re

from paper_2502_01277_amd.build import CSRC

# Barriers that nothing has read LDS before: the first operands of a launch have landed, then the loop over K steps begins.
PROLOGUES = {"conv.hip": 1, "conv_flow.h": 1, "conv3x3_mid.h": 1}


def test_barriers_wait_for_the_reads_of_the_stage_they_free():
    seen = 0
    for f in sorted(os.listdir(CSRC)):
        if not f.endswith((".h", ".hip")):
            continue
        lines = open(os.path.join(CSRC, f)).read().split("\n")
        bare = 0
        for i, line in enumerate(lines):
            if "__builtin_amdgcn_s_barrier()" not in line or line.lstrip().startswith("//"):
                continue
            # the wait stands right in front, or in the lambda `landed` that is called there
            waits = re.findall(r"s_waitcnt[^\"]*", "\n".join(lines[i - 7:i]))[-1:]
            if re.search(r"\blanded\(", lines[i - 1]):
                body = "\n".join(lines)
                waits = re.findall(r"s_waitcnt[^\"]*", re.search(r"auto landed = .*?\n    };", body, re.S).group(0))
            assert waits, (f, i + 1)
            seen += 1
            bare += any("lgkmcnt(0)" not in w for w in waits)
        assert bare == PROLOGUES.get(f, 0), (f, bare)
    assert seen >= 6
