"""Backwards cut into segments.  Where two passes of three are swept, dK's states are dV's transposed, written by the scan;
elsewhere all three are swept.  Every width and type, fewer and more segments than the scan has in flight, a short last
one, and infinities."""
import pytest
import torch

import paper_2307_14995_amd as ltn
from paper_2307_14995_amd import synth
from oracle import ltn_oracle as orc
from _helpers import TOL, check, force_plan, force_segs, gpu, mixed_decay

pytestmark = pytest.mark.gpu

BF, F32 = torch.bfloat16, torch.float32


@pytest.mark.parametrize("dtype", [BF, F32])
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
        assert ltn.ltn_attn_query_sweeps(Bt, H, N, D, dtype) == (2 if dtype == BF and D == 256 else 3)
        grads = ltn.ltn_attn_bwd(*gpu(q, k, v, g, decay))
    for n, x, r in zip(("dQ", "dK", "dV"), grads, orc.bwd_recurrent(q, k, v, g, decay)):
        check(n, x, r, TOL[dtype])


def ragged(D, segs):
    """Tokens of `segs` segments of more than D tokens, a multiple of 64, the last of D + 3."""
    return (segs - 1) * 64 * (D // 64 + 1) + D + 3


# chains x segments just past where three sweeps take a round of workgroups more than two, and up to the end of that round
PAIRED = [(D, segs, chains) for D in (64, 96, 128) for segs, chains in ((3, 30), (8, 12), (11, 9), (8, 16))] + \
         [(256, segs, chains) for segs, chains in ((3, 16), (8, 6), (11, 4), (8, 8))]


@pytest.mark.parametrize("D,segs,chains", PAIRED)
def test_gradients_from_two_sweeps_in_fp32(D, segs, chains):
    """The states lie in the outputs' rows; the last segment is the shorter one of a reversed axis."""
    N, H = ragged(D, segs), next(h for h in (3, 2) if chains % h == 0)
    Bt = chains // H
    q, k, v = synth.make_qkv(Bt, H, N, D, F32, 60 + segs)
    g = synth.make_do(Bt, H, N, D, F32, 60 + segs)
    decay = mixed_decay(H)
    with force_segs(segs):
        assert ltn.ltn_attn_query_plan(Bt, H, N, D, F32, 1)[1] == segs
        assert ltn.ltn_attn_query_sweeps(Bt, H, N, D, F32) == 2
        grads = ltn.ltn_attn_bwd(*gpu(q, k, v, g, decay))
    for n, x, r in zip(("dQ", "dK", "dV"), grads, orc.bwd_recurrent(q, k, v, g, decay)):
        check(n, x, r, TOL[F32])


@pytest.mark.parametrize("D,chains,dtype", [(64, 30, F32), (96, 30, F32), (128, 30, F32), (256, 16, F32), (256, 4, BF)])
@pytest.mark.parametrize("where", ["q", "g"])
def test_infinity_survives_segments_whose_decay_underflows(D, chains, dtype, where):
    """0.5^320 is zero in fp32: cut or whole, what an infinite query or output gradient of the last segment makes infinite
    in the earlier tokens' dK and dV stays so, and nothing else changes."""
    H, segs, N = 2, 3, 2 * 320 + 259
    decay = torch.tensor([0.5, 0.0])
    q, k, v = synth.make_qkv(chains // H, H, N, D, dtype, 77)
    g = synth.make_do(chains // H, H, N, D, dtype, 77)
    (q if where == "q" else g)[..., N - 4, 5] = float("inf")
    got = {}
    for n in (1, segs):
        with force_plan(0, n):
            assert ltn.ltn_attn_query_sweeps(chains // H, H, N, D, dtype) == (0 if n == 1 else 2)
            got[n] = [x.float().cpu()[:, 0] for x in ltn.ltn_attn_bwd(*gpu(q, k, v, g, decay))]
    for name, whole, cut in zip(("dQ", "dK", "dV"), got[1], got[segs]):
        assert torch.equal(whole.isnan(), cut.isnan()) and torch.equal(whole.isinf(), cut.isinf()), name
        bad = ~whole.isfinite()
        assert torch.equal(whole[bad].sign().nan_to_num(), cut[bad].sign().nan_to_num()), name
    # in both, of every earlier token: all features of the one; the feature's column of the other, sums over infinities
    column, rows = (1, 2) if where == "q" else (2, 1)
    assert got[segs][rows][..., :N - 4, :].isinf().all() and not got[segs][column][..., :N - 4, 5].isfinite().any()
    assert got[segs][column][..., 6:].isfinite().all()
