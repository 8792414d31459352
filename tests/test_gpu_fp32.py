"""GPU parity of the fp32 matrix-core pass at the edges of its tiles: every slice width and a
segmented plan (segment states kept in the output's rows) at ragged lengths, with a carried
state in both directions, against the fp64 oracle.

Tolerance: products and sums are fp32 throughout, so a result carries about sqrt(terms) roundings
of 2^-24 relative to its row's size: N + D <= 1000 terms give 2e-6; the bound is 1e-5."""
import pytest
import torch

import paper_2307_14995_amd as ltn
from paper_2307_14995_amd import synth
from oracle import ltn_oracle as orc
from _helpers import check, force_plan, gpu, mixed_decay

pytestmark = pytest.mark.gpu

TOL = 1e-5
PLANS = [(64, 64, 1), (64, 32, 1), (64, 64, 3), (96, 96, 1), (96, 32, 1), (96, 96, 3), (128, 128, 1), (128, 64, 1),
         (128, 32, 1), (128, 128, 3), (128, 32, 2), (256, 128, 1), (256, 64, 1), (256, 32, 1), (256, 128, 2)]


@pytest.mark.parametrize("D,dv,segs", PLANS)
@pytest.mark.parametrize("extra", [-1, 0, 1, 17])
def test_fp32_slices_and_segments(D, dv, segs, extra):
    N = 32 * 3 + extra if segs == 1 else segs * 64 * ((D + 63) // 64) + extra - 1
    Bt, H = 1, 3
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.float32, 300 + N)
    g = synth.make_do(Bt, H, N, D, torch.float32, 300 + N)
    decay = mixed_decay(H)
    kv0 = torch.randn(Bt, H, D, D, generator=torch.Generator().manual_seed(N)) / D
    with force_plan(dv, segs):
        assert ltn.ltn_attn_query_plan(Bt, H, N, D, torch.float32, 0)[0] == dv
        o, kv = ltn.ltn_attn_fwd(*gpu(q, k, v, decay), kv_in=kv0.cuda(), return_state=True)
        grads = ltn.ltn_attn_bwd(*gpu(q, k, v, g, decay))
    o_ref, kv_ref = orc.fwd_recurrent(q, k, v, decay, kv_in=kv0, return_state=True)
    check("O", o, o_ref, TOL)
    check("kv", kv, kv_ref, TOL)
    for n, x, r in zip(("dQ", "dK", "dV"), grads, orc.bwd_recurrent(q, k, v, g, decay)):
        check(n, x, r, TOL)


@pytest.mark.parametrize("Dk,Dv", [(256, 128), (128, 64)])
@pytest.mark.parametrize("segs,N", [(1, 33), (2, 515), (3, 800)])
def test_fp32_unequal_widths(Dk, Dv, segs, N):
    Bt, H = 1, 2
    q, k, v = synth.make_qkv_dkdv(Bt, H, N, Dk, Dv, torch.float32, 40 + N)
    g = synth.make_do(Bt, H, N, Dv, torch.float32, 40 + N)
    decay = mixed_decay(H)
    with force_plan(0, segs):
        o, kv = ltn.ltn_attn_fwd_dkdv(*gpu(q, k, v, decay), return_state=True)
        grads = ltn.ltn_attn_bwd_dkdv(*gpu(q, k, v, g, decay))
    o_ref, kv_ref = orc.fwd_recurrent_dkdv(q, k, v, decay, return_state=True)
    check("O", o, o_ref, TOL)
    check("kv", kv, kv_ref, TOL)
    for n, x, r in zip(("dQ", "dK", "dV"), grads, orc.bwd_recurrent_dkdv(q, k, v, g, decay)):
        check(n, x, r, TOL)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Bt,H,N", [(1, 2, 31), (1, 2, 777), (16, 16, 97)])
def test_fp32_gated_with_and_without_o(D, Bt, H, N):
    """Fused (many chains) and in two steps (few): the same bits whether O is stored or not."""
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.float32, 60 + N)
    u = synth.make_gate(Bt, H, N, D, torch.float32, 60 + N)
    decay = synth.decay_bench_rule(H)
    o_ref, y_ref = orc.fwd_gated(q, k, v, u, decay, eps=1e-6)
    o, y, kv = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6, return_state=True)
    _, y2, kv2 = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6, return_state=True, store_o=False)
    check("O", o, o_ref, TOL)
    check("Y", y, y_ref, 2 * TOL)          # the norm doubles a row's relative error at most
    assert torch.equal(y2, y) and torch.equal(kv2, kv)
