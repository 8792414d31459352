"""Chains cut into segments of 128 to 256 tokens by the library's own plan: the plan itself (host
only) and parity of forward, gated forward and gradients against the oracle at ragged lengths, the
state carried in and out.  Tolerances are the parity suite's: what bf16 operands and a state rounded
to bf16 for its products give, whatever the segment length."""
import pytest
import torch

import paper_2307_14995_amd as ltn
from paper_2307_14995_amd import synth
from oracle import ltn_oracle as orc
from _helpers import TOL, check, gpu, mixed_decay

BF = torch.bfloat16


def test_short_segment_plans_fit_one_round_and_the_scratch():
    for D in (64, 96, 128, 256):
        for call, passes in ((0, 1), (1, 3), (2, 1)):
            for chains in (1, 2, 3, 5, 8, 12, 20, 31, 40, 51, 64):
                for N in (65, 319, 640, 799, 800, 1000, 1537, 2000, 3001, 4097, 9999, 32768):
                    dv, segs = ltn.ltn_attn_query_plan(1, chains, N, D, BF, call)
                    assert segs == 1 or passes * chains * segs <= 256
                    need = ltn.ltn_attn_workspace_bytes(1, chains, N, D, 0, BF, call)
                    assert need >= (0 if segs == 1 else passes * chains * segs * D * D * 4)
                    assert need <= 16 << 20


def test_cuts_that_do_not_pay_are_not_taken():
    """Shapes whose forced cuts ran slower than the whole chain (5 .. 34 %), and neighbours where they pay."""
    def segs(chains, N, D, call):
        return ltn.ltn_attn_query_plan(1, chains, N, D, BF, call)[1]

    def scratch(chains, N, Dk, call):
        return ltn.ltn_attn_workspace_bytes_dkdv(1, chains, N, Dk, Dk // 2, BF, call)

    for chains in (1, 2, 4):
        assert segs(chains, 1537, 64, 1) == 1 and segs(chains, 1800, 64, 1) == 1 and segs(chains, 2500, 64, 1) > 4
    for chains in (40, 51):
        assert segs(chains, 800, 64, 2) == 1 and segs(chains, 1290, 64, 2) > 3
    assert segs(51, 800, 128, 2) == 1 and segs(24, 800, 128, 2) == 5
    # 1290 tokens in five segments are four of 320 and one of 10
    for chains in (10, 12, 16):
        assert segs(chains, 1290, 96, 0) == 1 and segs(chains, 1537, 96, 0) > 1
    assert segs(4, 1290, 256, 1) == 1 and segs(4, 1290, 256, 0) == 5
    for N in (1537, 1800, 2000):
        assert scratch(64, N, 128, 0) == 0 and scratch(64, N, 128, 1) == 0 and scratch(8, N, 128, 0) > 0
    assert scratch(48, 1290, 128, 0) == 0 and scratch(4, 1290, 256, 0) > 0


CASES = [("gated", 1, 3, 800, 128), ("gated", 1, 4, 1001, 64), ("gated", 2, 3, 1087, 128), ("fwd", 1, 4, 1999, 128),
         ("fwd", 2, 4, 2049, 64), ("bwd", 1, 4, 2050, 64), ("bwd", 1, 3, 3011, 128), ("fwd", 1, 2, 1345, 256), ("bwd", 1, 2, 1999, 96)]


@pytest.mark.gpu
@pytest.mark.parametrize("call,Bt,H,N,D", CASES)
def test_short_segments_match_the_oracle(call, Bt, H, N, D):
    segs = ltn.ltn_attn_query_plan(Bt, H, N, D, BF, ("fwd", "bwd", "gated").index(call))[1]
    assert segs > 1 and N / segs < 512
    q, k, v = synth.make_qkv(Bt, H, N, D, BF, 900 + N)
    g = synth.make_do(Bt, H, N, D, BF, 900 + N)
    decay = mixed_decay(H)
    kv0 = torch.randn(Bt, H, D, D, generator=torch.Generator().manual_seed(N)) / D
    if call == "bwd":
        for n, x, r in zip(("dQ", "dK", "dV"), ltn.ltn_attn_bwd(*gpu(q, k, v, g, decay)),
                           orc.bwd_recurrent(q, k, v, g, decay)):
            check(n, x, r, TOL[BF])
        return
    o_ref, kv_ref = orc.fwd_recurrent(q, k, v, decay, kv_in=kv0, return_state=True)
    if call == "fwd":
        o, kv = ltn.ltn_attn_fwd(*gpu(q, k, v, decay), kv_in=kv0.cuda(), return_state=True)
        check("O", o, o_ref, TOL[BF])
    else:
        _, y, kv = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, g, decay), eps=1e-6, kv_in=kv0.cuda(), return_state=True,
                                          store_o=False)
        ref = torch.as_tensor(o_ref)
        ref = ref / torch.sqrt((ref * ref).mean(-1, keepdim=True) + 1e-6) * g.double()
        check("y", y, ref.numpy(), TOL[BF])
    check("kv", kv, kv_ref, TOL[BF])


@pytest.mark.gpu
@pytest.mark.parametrize("Dk,N", [(256, 1537), (256, 1290), (128, 2001)])
def test_short_segments_of_unequal_widths(Dk, N):
    Bt, H, Dv = 1, 3, Dk // 2
    assert ltn.ltn_attn_workspace_bytes_dkdv(Bt, H, N, Dk, Dv, BF, 0) > 0
    q, k, v = synth.make_qkv_dkdv(Bt, H, N, Dk, Dv, BF, 950 + N)
    g = synth.make_do(Bt, H, N, Dv, BF, 950 + N)
    decay = mixed_decay(H)
    o, kv = ltn.ltn_attn_fwd_dkdv(*gpu(q, k, v, decay), return_state=True)
    o_ref, kv_ref = orc.fwd_recurrent_dkdv(q, k, v, decay, return_state=True)
    check("O", o, o_ref, TOL[BF])
    check("kv", kv, kv_ref, TOL[BF])
    for n, x, r in zip(("dQ", "dK", "dV"), ltn.ltn_attn_bwd_dkdv(*gpu(q, k, v, g, decay)),
                       orc.bwd_recurrent_dkdv(q, k, v, g, decay)):
        check(n, x, r, TOL[BF])


@pytest.mark.gpu
@pytest.mark.parametrize("H,N", [(3, 1), (3, 512), (70, 511), (3, 1000)])
def test_fused_gated_forward_that_stores_o(H, N):
    # heads of 64 features: short, or cut into segments
    q, k, v = synth.make_qkv(1, H, N, 64, BF, 970 + N)
    u = synth.make_gate(1, H, N, 64, BF, 970 + N)
    decay = mixed_decay(H)
    o_ref, y_ref = orc.fwd_gated(q, k, v, u, decay, eps=1e-6)
    o, y = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6)
    check("O", o, o_ref, TOL[BF])
    check("Y", y, y_ref, TOL[BF])
