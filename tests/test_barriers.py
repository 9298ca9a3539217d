"""Every workgroup barrier of the kernels waits for the wave's own LDS accesses.

A wave that has issued an LDS read and crosses a bare ``s_barrier`` may still have the read in flight when another wave,
past the same barrier, overwrites the location.  Results cannot show that a schedule happens to hide this, so the
sources are held to the rule: ``s_barrier`` is written only behind ``s_waitcnt lgkmcnt(0)`` in the same statement
(``__syncthreads()`` carries its own wait).
"""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_14568_amd", "csrc")


def test_barriers_wait_for_lds():
    found, bare = 0, []
    for name in sorted(os.listdir(CSRC)):
        for n, line in enumerate(open(os.path.join(CSRC, name)), 1):
            code = re.sub(r"lds_barrier|//.*", "", line)
            found += code.count("s_barrier")
            if "s_barrier" in code.replace(r"s_waitcnt lgkmcnt(0)\n\ts_barrier", ""):
                bare.append("%s:%d" % (name, n))
    assert found > 0 and not bare, bare
