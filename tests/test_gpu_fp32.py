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


def cut_length(D, segs, extra):
    """A length that the kernel cuts `segs` ways, the last segment D + extra tokens long (every segment holds
    a D x D state in its output rows): the others are the multiple of 64 above that."""
    return (segs - 1) * (64 * ((D + 63) // 64) + (64 if D % 64 == 0 else 0)) + D + extra


@pytest.mark.parametrize("D,dv,segs", PLANS)
@pytest.mark.parametrize("extra", [-1, 0, 1, 17])
def test_fp32_slices_and_segments(D, dv, segs, extra):
    N = 32 * 3 + extra if segs == 1 else cut_length(D, segs, extra + 5)
    Bt, H = 1, 3
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.float32, 300 + N)
    g = synth.make_do(Bt, H, N, D, torch.float32, 300 + N)
    decay = mixed_decay(H)
    kv0 = torch.randn(Bt, H, D, D, generator=torch.Generator().manual_seed(N)) / D
    with force_plan(dv, segs):
        for call in (0, 1):
            assert ltn.ltn_attn_query_plan(Bt, H, N, D, torch.float32, call) == (dv, segs)
        o, kv = ltn.ltn_attn_fwd(*gpu(q, k, v, decay), kv_in=kv0.cuda(), return_state=True)
        grads = ltn.ltn_attn_bwd(*gpu(q, k, v, g, decay))
    o_ref, kv_ref = orc.fwd_recurrent(q, k, v, decay, kv_in=kv0, return_state=True)
    check("O", o, o_ref, TOL)
    check("kv", kv, kv_ref, TOL)
    for n, x, r in zip(("dQ", "dK", "dV"), grads, orc.bwd_recurrent(q, k, v, g, decay)):
        check(n, x, r, TOL)


@pytest.mark.parametrize("D,dv,segs", PLANS)
@pytest.mark.parametrize("missing", [1, 33])
def test_fp32_too_short_to_cut(D, dv, segs, missing):
    """A last segment with fewer than D tokens has no room for its state: fewer segments, the same results."""
    N = cut_length(D, segs, -missing) if segs > 1 else 2 * D - missing
    Bt, H = 1, 3
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.float32, 350 + N)
    decay = mixed_decay(H)
    with force_plan(dv, segs):
        assert ltn.ltn_attn_query_plan(Bt, H, N, D, torch.float32, 0)[1] <= segs
        o, kv = ltn.ltn_attn_fwd(*gpu(q, k, v, decay), return_state=True)
    o_ref, kv_ref = orc.fwd_recurrent(q, k, v, decay, return_state=True)
    check("O", o, o_ref, TOL)
    check("kv", kv, kv_ref, TOL)


# (segs, N) of a width pair: whole, and cut with a ragged last segment in both shapes of its passes (the
# states of either take Dk x Dv, in rows of Dv or Dk)
@pytest.mark.parametrize("Dk,Dv", [(256, 128), (128, 64)])
@pytest.mark.parametrize("segs", [1, 2, 3])
def test_fp32_unequal_widths(Dk, Dv, segs):
    N = 33 if segs == 1 else cut_length(Dk, segs, 13)
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


def gated_reference(q, k, v, u, decay, kv0):
    o, kv = orc.fwd_recurrent(q, k, v, decay, kv_in=kv0, return_state=True)
    return o, orc.gate_fwd(o, u, 1e-6), kv


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("extra", [0, 5, 17])
def test_fp32_fused_gated_pass_on_segments(D, extra):
    """The fused epilogue with the segments' states in o's rows (stored) or y's (not): the same bits, the
    state carried in, out and in place, nothing written beside the outputs."""
    Bt, H, segs = 1, 3, 3
    N = cut_length(D, segs, extra)
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.float32, 80 + N)
    u = synth.make_gate(Bt, H, N, D, torch.float32, 80 + N)
    decay = torch.tensor([1.0, 0.5, 0.98])
    kv0 = torch.randn(Bt, H, D, D, generator=torch.Generator().manual_seed(N)) / D
    o_ref, y_ref, kv_ref = gated_reference(q, k, v, u, decay, kv0)
    guard = 1024                           # floats on each side of an output

    def guarded(n):
        raw = torch.full((n + 2 * guard,), 7.0, device="cuda")
        return raw, raw[guard:guard + n]

    args = gpu(q, k, v, u, decay)
    with force_plan(D, segs):              # the plain forward at full width too: fused is the choice
        assert ltn.ltn_attn_query_plan(Bt, H, N, D, torch.float32, 2) == (D, segs)
        raws, outs = zip(*(guarded(n) for n in (q.numel(), q.numel(), kv0.numel())))
        o, y, kv = outs[0].view_as(q), outs[1].view_as(q), outs[2].view_as(kv0)
        ltn.ltn_attn_fwd_gated(*args, eps=1e-6, kv_in=kv0.cuda(), out=o, y_out=y, kv_out=kv)
        raw2, y2 = guarded(q.numel())
        state = kv0.cuda()
        ltn.ltn_attn_fwd_gated(*args, eps=1e-6, kv_in=state, store_o=False, y_out=y2.view_as(q), kv_out=state)
    check("O", o, o_ref, TOL)
    check("Y", y, y_ref, 2 * TOL)          # the norm doubles a row's relative error at most
    check("kv", kv, kv_ref, TOL)
    assert torch.equal(y2, y.flatten()) and torch.equal(state, kv)
    for raw in (*raws, raw2):
        assert bool((raw[:guard] == 7.0).all()) and bool((raw[-guard:] == 7.0).all())


def test_fp32_gated_call_of_the_385m_shape_runs_fused_on_segments():
    Bt, H, N, D = 4, 8, 2048, 128
    assert ltn.ltn_attn_query_plan(Bt, H, N, D, torch.float32, 2) == (128, 8)
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.float32, 91)
    u = synth.make_gate(Bt, H, N, D, torch.float32, 91)
    decay = synth.decay_bench_rule(H)
    o_ref, y_ref, kv_ref = gated_reference(q, k, v, u, decay, torch.zeros(Bt, H, D, D))
    o, y, kv = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6, return_state=True)
    check("O", o, o_ref, TOL)
    check("Y", y, y_ref, 2 * TOL)
    check("kv", kv, kv_ref, TOL)


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


@pytest.mark.parametrize("Bt,H,N", [(29, 3, 1), (29, 3, 33), (29, 3, 64), (29, 9, 97)])
def test_fp32_two_workgroups_a_unit(Bt, H, N):
    """Heads of 64 features with more than 256 workgroups (3 x 87 and 261 chains): the four-wave instance, both
    directions, the state carried."""
    D = 64
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.float32, 700 + N)
    g = synth.make_do(Bt, H, N, D, torch.float32, 700 + N)
    decay = mixed_decay(H)
    kv0 = torch.randn(Bt, H, D, D, generator=torch.Generator().manual_seed(N)) / D
    with force_plan(D, 1):
        o, kv = ltn.ltn_attn_fwd(*gpu(q, k, v, decay), kv_in=kv0.cuda(), return_state=True)
        grads = ltn.ltn_attn_bwd(*gpu(q, k, v, g, decay))
    o_ref, kv_ref = orc.fwd_recurrent(q, k, v, decay, kv_in=kv0, return_state=True)
    check("O", o, o_ref, TOL)
    check("kv", kv, kv_ref, TOL)
    for n, x, r in zip(("dQ", "dK", "dV"), grads, orc.bwd_recurrent(q, k, v, g, decay)):
        check(n, x, r, TOL)
