"""Rules of the kernel sources that no run shows: what a break of them does depends on the registers that the
compiler happens to choose."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_22718_amd", "csrc")


def test_no_value_is_read_from_another_lanes_register():
    """v_readlane reads its lane whether or not it is active, and in a divergent loop a spill reload or a
    register copy leaves the inactive lanes stale: wave-uniform values go through scalar registers, scalar
    loads or LDS.  (readfirstlane takes an active lane.)"""
    for name in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, name)) as f:
            code = re.sub(r"//[^\n]*", "", f.read())
        assert "__builtin_amdgcn_readlane" not in code, name
