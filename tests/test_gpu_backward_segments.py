"""Backwards cut into segments: dK's states are dV's transposed, written by the scan.  Every width, fewer and more segments
than the scan has in flight, a short last one."""
import pytest
import torch

import paper_2307_14995_amd as ltn
from paper_2307_14995_amd import synth
from oracle import ltn_oracle as orc
from _helpers import TOL, check, force_segs, gpu, mixed_decay

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D", [64, 96, 128, 256])
@pytest.mark.parametrize("segs", [2, 8, 11])
def test_gradients(D, segs, dtype):
    Bt, H = 1, 3
    length = -(-D // 64) * 64                      # fp32 segments hold a whole state in their rows
    N = (segs - 1) * length + D + 3
    if segs * length < N:
        N = segs * length
    q, k, v = synth.make_qkv(Bt, H, N, D, dtype, 40 + segs)
    g = synth.make_do(Bt, H, N, D, dtype, 40 + segs)
    decay = mixed_decay(H)
    with force_segs(segs):
        assert ltn.ltn_attn_query_plan(Bt, H, N, D, dtype, 1)[1] == segs
        grads = ltn.ltn_attn_bwd(*gpu(q, k, v, g, decay))
    for n, x, r in zip(("dQ", "dK", "dV"), grads, orc.bwd_recurrent(q, k, v, g, decay)):
        check(n, x, r, TOL[dtype])
