"""Counted waits (`s_waitcnt vmcnt(n)`, n > 0) hold only where every load that they leave in flight is written out in the source."""
import os
import re

import pytest

from paper_2412_12094_amd import build


@pytest.mark.parametrize("name", ["fwd_bf16.hip", "bwd_dq.h"])
def test_no_counted_wait_over_loads_that_the_compiler_issues(name):
    """These kernels fetch query rows with ordinary loads, which the compiler may merge, drop or move."""
    with open(os.path.join(build.CSRC, name)) as f:
        waits = re.findall(r"vmcnt\(([^)]*)\)", f.read())
    assert waits and set(waits) == {"0"}
