"""Which fp32 backwards of 128 features are cut into segments: shapes whose times as whole chains and cut were both
measured (us: whole or the plan before, and the other)."""
import pytest
import torch

import paper_2307_14995_amd as ltn

# (chains, N, value columns, segments, us of this plan, us of the other one that the estimate comes near to)
MEASURED = [
    (16, 1024, 32, 1, 67, 75), (26, 1024, 64, 1, 101, 119), (32, 1024, 64, 1, 102, 120), (18, 1300, 32, 1, 84, 97),
    (26, 1500, 128, 3, 136, 158), (56, 1500, 128, 1, 240, 269), (26, 1999, 128, 3, 180, 198), (53, 2048, 128, 1, 327, 365),
    (18, 2048, 32, 1, 129, 143), (64, 4096, 128, 1, 654, 693), (12, 8192, 128, 7, 300, 324), (64, 8192, 128, 1, 1307, 1368),
    (32, 2048, 128, 8, 198, 222), (22, 2500, 128, 10, 194, 207), (24, 8192, 128, 10, 552, 593), (23, 16384, 128, 10, 1068, 1127),
    (52, 8192, 128, 6, 1242, 1298), (52, 16384, 128, 6, 2410, 2611),
]


@pytest.mark.parametrize("chains,N,dv,segs,us,other", MEASURED)
def test_plan_is_the_faster_one(chains, N, dv, segs, us, other):
    assert us < other
    assert ltn.ltn_attn_query_plan(1, chains, N, 128, torch.float32, 1) == (dv, segs)
