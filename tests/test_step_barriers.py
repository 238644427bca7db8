"""The step's workgroup barriers on the way a chained launch's idle groups stand beside: each of the
list StepBarrier once, and no other, or those groups would wait for a barrier that never comes."""

import os
import re

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_10118_amd", "csrc",
                   "kernels.hip")


def test_step_body_passes_each_listed_barrier_once():
    with open(SRC) as f:
        text = f.read()
    names = [n.strip() for n in re.search(r"enum StepBarrier \{([^}]*)\}", text).group(1).split(",")]
    assert names[-1] == "STEP_BARRIERS" and len(names) > 1
    start = text.index("__device__ __forceinline__ void step_body(")
    body = text[start:text.index("// ---- deep hierarchies", start)]
    assert re.findall(r"step_barrier<(\w+)>\(\);", body) == names[:-1]
    assert "__syncthreads" not in body and "s_barrier" not in body
