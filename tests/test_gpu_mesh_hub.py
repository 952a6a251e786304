"""A vertex with far more incident corners than any row may have (the highest
number of a fan, which pc_create's own limit on edges at their lower end does
not see): the context is made without delay and every assembly is refused."""
import time

import pytest

from gpu_helpers import random_velocity, require_gpu, to_dev
from test_gpu_wide_rows import fan_cloth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [255, 256, 257, 30000])   # 2 n corners at the centre; 512 are the most a row may have
def test_hub(n):
    torch = require_gpu()
    from paper_2008_00409_amd import binding as B
    c = fan_cloth(n)
    x, v = to_dev(torch, c.x0), to_dev(torch, random_velocity(c))
    B.Context.from_cloth(fan_cloth(8)).close()   # what the first context of a process loads
    t0 = time.perf_counter()
    ctx = B.Context.from_cloth(c)
    try:
        # 60,000 corners: sorted by rank they are 2.25e8 steps of 16 lanes, tens of
        # seconds; copied they are 3,750
        assert time.perf_counter() - t0 < 2.0
        for _ in range(2):
            b = ctx.cloth_assemble(x, v, "f32")
            with pytest.raises(B.PclothError, match="PC_ERR_CAPACITY"):
                ctx.cloth_pcg_solve(b)
    finally:
        ctx.close()
