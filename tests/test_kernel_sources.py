"""Rules of the kernel sources that no run on the GPU can show broken."""
from __future__ import annotations

import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_0710_1272_amd", "csrc")


def test_no_workgroup_library_reduction_in_the_bead_step():
    """In the one-launch step the bead step runs with part of its workgroup gone; the device
    library's workgroup reductions are specified for all threads of the workgroup."""
    with open(os.path.join(CSRC, "md_bead.hpp")) as fh:
        code = re.sub(r"//[^\n]*", "", fh.read())
    assert not re.findall(r"__syncthreads_(?:or|and|count)\b", code)


def test_one_launch_step_sets_no_attribute_when_it_launches():
    """The launch may fall inside a graph capture: lb_init sets the kernel's LDS attribute."""
    with open(os.path.join(CSRC, "md_bead.hpp")) as fh:
        code = fh.read()
    launch = code[code.index("launch_step_one_t("):code.index("launch_step_one_g(")]
    assert "hipLaunchKernelGGL" in launch and "hipFuncSetAttribute" not in launch
