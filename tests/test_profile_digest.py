"""The digest that marks counters as stale covers every file of this repository that the step
kernels include."""
import os
import re

from paper_1412_6426_amd.calib import profile_summary as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DIRS = (os.path.join(ROOT, "paper_1412_6426_amd", "csrc"), os.path.join(ROOT, "include"))


def test_digest_covers_the_headers_that_the_kernels_include():
    seen, todo = set(), [P.KERNEL_SRC]
    while todo:
        f = todo.pop()
        if f in seen:
            continue
        seen.add(f)
        for name in re.findall(r'#include "([^"]+)"', open(f).read()):
            todo += [p for p in (os.path.join(d, name) for d in DIRS) if os.path.exists(p)]
    assert seen == {P.KERNEL_SRC, *P.KERNEL_HEADERS}
