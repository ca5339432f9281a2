"""CPU: barriers written by hand in the kernels also wait for the wavefront's own LDS accesses, because what follows them overwrites what was read
before: the compiler orders the instructions around a barrier, but the data of a read only have to be there where they are used.
"""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2508_18376_amd", "csrc")
# its callers pin the matrix instructions that use what was read in front of it (sched_barrier), and it must not wait for the next stage's reads
PINNED = {("gemm_mfma.hip", "block_barrier")}


def test_hand_written_barriers_wait_for_lds():
    found = 0
    for name in sorted(os.listdir(CSRC)):
        for line in open(os.path.join(CSRC, name)):
            if "s_barrier" not in line or "asm" not in line:
                continue
            found += 1
            fn = re.search(r"void (\w+)\(", line)
            if (name, fn and fn.group(1)) in PINNED:
                continue
            assert re.search(r"s_waitcnt lgkmcnt\(0\)\\n\\ts_barrier", line), (name, line.strip())
    assert found >= 3
