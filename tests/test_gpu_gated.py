"""GPU parity of the gated, normalised output (Sec. 3.1.2 Eq. 3 with the SimpleRMSNorm of
Sec. 3.1.3 per head): the fused forward epilogue and the stand-alone gate kernels, through
the C ABI, against the fp64 oracle on the same seeded inputs."""
import numpy as np
import pytest
import torch

import paper_2307_14995_amd as ltn
from paper_2307_14995_amd import synth
from oracle import ltn_oracle as orc
from _helpers import TOL_ROW, check, check_rows, dev, force_plan, gpu, mixed_decay

pytestmark = pytest.mark.gpu

TOL = {torch.float32: 1e-4, torch.bfloat16: 1e-2}


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("eps", [0.0, 1e-5])
def test_gate_rows_forward_backward(dtype, D, eps):
    rows = 4099                               # not a multiple of any rows-per-workgroup step
    g = torch.Generator().manual_seed(900 + D)
    x = (torch.randn(rows, D, generator=g) * 0.7).to(dtype)
    u = torch.randn(rows, D, generator=g).to(dtype)
    dy = torch.randn(rows, D, generator=g).to(dtype)
    xd, ud, dyd = gpu(x, u, dy)
    y = ltn.ltn_gate_fwd(xd, ud, eps)
    dx, du = ltn.ltn_gate_bwd(xd, ud, dyd, eps)
    tol = TOL[dtype]
    assert orc.rel_l2(y, orc.gate_fwd(x, u, eps)) <= tol
    dx_ref, du_ref = orc.gate_bwd(x, u, dy, eps)
    assert orc.rel_l2(dx, dx_ref) <= tol
    assert orc.rel_l2(du, du_ref) <= tol
    # row-wise too: no row may be off (catches a reduction that mixes neighbouring rows)
    yr = orc.gate_fwd(x, u, eps)
    row_err = np.linalg.norm(y.double().cpu().numpy() - yr, axis=1) / np.linalg.norm(yr, axis=1)
    assert row_err.max() <= 4 * tol


def test_gate_rows_empty_and_errors():
    x = torch.zeros(0, 128, dtype=torch.bfloat16, device=dev())
    assert ltn.ltn_gate_fwd(x, x).shape == (0, 128)
    a = torch.ones(4, 128, dtype=torch.bfloat16, device=dev())
    with pytest.raises(ltn.LtnError):
        ltn.ltn_gate_fwd(a, a, out=a)                     # output aliases an input
    with pytest.raises(ltn.LtnError):
        ltn.ltn_gate_fwd(a[:, :80].contiguous(), a[:, :80].contiguous())   # D = 80 not built
    with pytest.raises(ltn.LtnError):
        ltn.ltn_gate_fwd(a, a, eps=-1.0)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N", [1, 63, 64, 65, 200, 517])
def test_bf16_forward_gated_ragged(D, N):
    Bt, H = 1, 3
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.bfloat16, 400 + N)
    u = synth.make_gate(Bt, H, N, D, torch.bfloat16, 400 + N)
    decay = mixed_decay(H)
    o_ref, y_ref = orc.fwd_gated(q, k, v, u, decay, eps=1e-6)
    _, kv_ref = orc.fwd_recurrent(q, k, v, decay, return_state=True)
    o, y, kv = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6, return_state=True)
    check("O", o, o_ref, 1e-2)
    check("Y", y, y_ref, 1e-2)
    check("kv", kv, kv_ref, 1e-2)
    # inference form: the attention output is not stored (always the fused epilogue)
    o2, y2 = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6, store_o=False)
    assert o2 is None
    check("Y (o not stored)", y2, y_ref, 1e-2)
    # and O is what the plain forward at full width gives
    assert orc.rel_l2(o, ltn.ltn_attn_fwd(*gpu(q, k, v, decay))) <= 1e-2


@pytest.mark.parametrize("D,block", [(64, 16), (64, 64), (128, 32)])
@pytest.mark.parametrize("N", [1, 37, 130])
def test_fp32_forward_gated(D, block, N):
    Bt, H = 2, 3
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.float32, 500 + N)
    u = synth.make_gate(Bt, H, N, D, torch.float32, 500 + N)
    decay = mixed_decay(H)
    o_ref, y_ref = orc.fwd_gated(q, k, v, u, decay, eps=0.0)
    o, y = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=0.0, block=block)
    check("O", o, o_ref, 1e-4)
    check("Y", y, y_ref, 1e-4)
    _, y2 = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=0.0, block=block, store_o=False)
    assert torch.equal(y2, y)


def test_bf16_forward_gated_continues_a_state():
    Bt, H, N, D = 2, 4, 300, 128
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.bfloat16, 43)
    u = synth.make_gate(Bt, H, N, D, torch.bfloat16, 43)
    decay = mixed_decay(H)
    cut = 131
    qd, kd, vd, ud, dd = gpu(q, k, v, u, decay)
    _, kv1 = ltn.ltn_attn_fwd(qd[:, :, :cut].contiguous(), kd[:, :, :cut].contiguous(),
                              vd[:, :, :cut].contiguous(), dd, return_state=True)
    _, y2 = ltn.ltn_attn_fwd_gated(qd[:, :, cut:].contiguous(), kd[:, :, cut:].contiguous(),
                                   vd[:, :, cut:].contiguous(), ud[:, :, cut:].contiguous(), dd,
                                   eps=1e-6, kv_in=kv1)
    _, y_ref = orc.fwd_gated(q, k, v, u, decay, eps=1e-6)
    check("Y tail", y2, y_ref[:, :, cut:], 1e-2)


def test_bf16_forward_gated_many_chains_fused_with_o():
    """>= 192 chains: the fused epilogue also when O is stored; both outputs against the oracle."""
    Bt, H, N, D = 8, 25, 70, 128             # 200 chains, ragged N
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.bfloat16, 45)
    u = synth.make_gate(Bt, H, N, D, torch.bfloat16, 45)
    decay = synth.decay_bench_rule(H)
    o_ref, y_ref = orc.fwd_gated(q, k, v, u, decay, eps=1e-6)
    o, y = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6)
    check("O", o, o_ref, 1e-2)
    check("Y", y, y_ref, 1e-2)
    _, y2 = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6, store_o=False)
    assert torch.equal(y2, y)                # same kernel, same bits


@pytest.mark.parametrize("segs,N", [(3, 517), (5, 1000)])
def test_bf16_forward_gated_segmented(segs, N):
    """The fused epilogue on chains cut into segments (forced), with an initial state."""
    Bt, H, D = 1, 3, 128
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.bfloat16, 460 + N)
    u = synth.make_gate(Bt, H, N, D, torch.bfloat16, 460 + N)
    kv0 = torch.randn(Bt, H, D, D, generator=torch.Generator().manual_seed(N)) * 0.1
    decay = mixed_decay(H)
    o_ref, y_ref = orc.fwd_gated(q, k, v, u, decay, eps=1e-6, kv_in=kv0)
    _, kv_ref = orc.fwd_recurrent(q, k, v, decay, kv_in=kv0, return_state=True)
    with force_plan(segs=segs):
        assert ltn.ltn_attn_workspace_bytes(Bt, H, N, D, 0, torch.bfloat16, 2) > 0
        _, y, kv = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6, kv_in=kv0.to(dev()),
                                          return_state=True, store_o=False)
    check("Y", y, y_ref, 1e-2)
    check("kv", kv, kv_ref, 1e-2)


def test_bf16_forward_gated_few_long_chains_by_default():
    Bt, H, N, D = 1, 4, 4096 + 50, 128       # 4 chains: cut 8 ways by the library's own rule, the fused form and
    # the plain forward (+ gate kernel, the form taken when O is stored) alike; the query covers both
    assert ltn.ltn_attn_query_plan(Bt, H, N, D, torch.bfloat16, 2) == (128, 8)
    assert ltn.ltn_attn_workspace_bytes(Bt, H, N, D, 0, torch.bfloat16, 2) == 8 * Bt * H * D * D * 4
    assert ltn.ltn_attn_workspace_bytes(Bt, H, N, D, 0, torch.bfloat16, 0) == 8 * Bt * H * D * D * 4
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.bfloat16, 49)
    u = synth.make_gate(Bt, H, N, D, torch.bfloat16, 49)
    decay = synth.decay_bench_rule(H)
    o_ref, y_ref = orc.fwd_gated(q, k, v, u, decay, eps=1e-6)
    o, y = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6)      # training form: plain forward + gate kernel
    _, y2 = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6, store_o=False)   # fused, segmented
    check("O", o, o_ref, 1e-2)
    check("Y", y, y_ref, 1e-2)
    check("Y (fused)", y2, y_ref, 1e-2)


def test_training_chain_through_the_gate():
    """fwd_gated (stores O) -> gate_bwd -> attn_bwd.  Every kernel is held to the 1e-2 bound
    against the oracle applied to the inputs that kernel really saw (the stored bf16 O, the
    stored bf16 dO); the chain end to end, whose error also holds the oracle's own sensitivity
    to those two roundings (the norm's derivative amplifies an error in O about twofold), is
    held to 2e-2."""
    Bt, H, N, D = 2, 3, 160, 128
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.bfloat16, 47)
    u = synth.make_gate(Bt, H, N, D, torch.bfloat16, 47)
    dy = synth.make_do(Bt, H, N, D, torch.bfloat16, 47)
    decay = synth.decay_bench_rule(H)
    qd, kd, vd, ud, dyd, dd = gpu(q, k, v, u, dy, decay)
    o, y = ltn.ltn_attn_fwd_gated(qd, kd, vd, ud, dd, eps=1e-6)
    d_o, d_u = ltn.ltn_gate_bwd(o, ud, dyd, eps=1e-6)
    dq, dk, dv = ltn.ltn_attn_bwd(qd, kd, vd, d_o, dd)
    # kernel by kernel, on the tensors each kernel was handed
    o_ref, y_ref = orc.fwd_gated(q, k, v, u, decay, eps=1e-6)
    check("O", o, o_ref, 1e-2)
    check("Y", y, y_ref, 1e-2)
    do_k, du_k = orc.gate_bwd(o.cpu(), u, dy, eps=1e-6)
    check("dO | stored O", d_o, do_k, 1e-2)
    check("dU | stored O", d_u, du_k, 1e-2)
    for n, x, r in zip(("dQ", "dK", "dV"), (dq, dk, dv), orc.bwd_recurrent(q, k, v, d_o.cpu(), decay)):
        check(n + " | stored dO", x, r, 1e-2)
    # end to end against the oracle's own chain
    do_ref, du_ref = orc.gate_bwd(o_ref, u, dy, eps=1e-6)
    check("dO", d_o, do_ref, 2e-2)
    check("dU", d_u, du_ref, 1e-2)
    for n, x, r in zip(("dQ", "dK", "dV"), (dq, dk, dv), orc.bwd_recurrent(q, k, v, do_ref, decay)):
        check(n, x, r, 2e-2)


def test_forward_gated_full_size_every_chain():
    """The 7B-shaped workload in the launch configuration the report times: every chain's Y
    against the oracle, slice by slice and token by token."""
    w = synth.CONFIGS["cfg3_7b"]
    q, k, v = synth.make_qkv(w.Bt, w.H, w.N, w.D, w.dtype, w.seed)
    u = synth.make_gate(w.Bt, w.H, w.N, w.D, w.dtype, w.seed)
    decay = synth.decay_bench_rule(w.H)
    _, y = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6, store_o=False)
    y = y.cpu()
    worst = 0.0
    for b in range(w.Bt):
        sl = slice(b, b + 1)
        o_ref = orc.fwd_recurrent(q[sl], k[sl], v[sl], decay)
        y_ref = orc.gate_fwd(o_ref, u[sl], 1e-6)
        check(f"Y[{b}]", y[sl], y_ref, 1e-2)
        worst = max(worst, check_rows(f"Y[{b}] rows", y[sl], y_ref, TOL_ROW[w.dtype]))
    print(f"gated cfg3: worst per-token error {worst:.2e}")


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D", [96, 256])
def test_gated_other_head_dims(dtype, D):
    """96 and 256 features: the gate kernels on rows, and the gated forward in the form every
    width and dtype has (plain forward, then the epilogue on the stored attention output)."""
    tol = TOL[dtype]
    rows = 1031
    g = torch.Generator().manual_seed(940 + D)
    x = (torch.randn(rows, D, generator=g) * 0.7).to(dtype)
    u = torch.randn(rows, D, generator=g).to(dtype)
    dy = torch.randn(rows, D, generator=g).to(dtype)
    xd, ud, dyd = gpu(x, u, dy)
    y = ltn.ltn_gate_fwd(xd, ud, 1e-6)
    dx, du = ltn.ltn_gate_bwd(xd, ud, dyd, 1e-6)
    yr = orc.gate_fwd(x, u, 1e-6)
    dx_ref, du_ref = orc.gate_bwd(x, u, dy, 1e-6)
    assert orc.rel_l2(y, yr) <= tol and orc.rel_l2(dx, dx_ref) <= tol and orc.rel_l2(du, du_ref) <= tol
    row_err = np.linalg.norm(y.double().cpu().numpy() - yr, axis=1) / np.linalg.norm(yr, axis=1)
    assert row_err.max() <= 2 * tol           # no row may be off (a reduction that mixes neighbouring rows)
    Bt, H, N = 2, 3, 150
    q, k, v = synth.make_qkv(Bt, H, N, D, dtype, 950 + D)
    ug = synth.make_gate(Bt, H, N, D, dtype, 950 + D)
    decay = mixed_decay(H)
    o, yy = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, ug, decay), eps=1e-6)
    o_ref = orc.fwd_recurrent(q, k, v, decay)
    check("O", o, o_ref, tol)
    check("Y | stored O", yy, orc.gate_fwd(o.cpu(), ug, 1e-6), tol)
    check("Y", yy, orc.gate_fwd(o_ref, ug, 1e-6), 2 * tol)      # end to end: one stored rounding deep
    if D == 96 and dtype == torch.bfloat16:      # a workgroup holds all 96 columns of a row: the fused form exists
        _, y2 = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, ug, decay), eps=1e-6, store_o=False)
        check("Y (fused)", y2, orc.gate_fwd(o_ref, ug, 1e-6), tol)
    else:
        with pytest.raises(ltn.LtnError):
            ltn.ltn_attn_fwd_gated(*gpu(q, k, v, ug, decay), eps=1e-6, store_o=False)


@pytest.mark.parametrize("N,segs", [(1, 0), (63, 0), (65, 0), (333, 0), (517, 3), (1000, 5)])
def test_bf16_forward_gated_96_features(N, segs):
    """The fused epilogue on heads of 96 features (all 96 value columns in one workgroup), ragged
    lengths, with an initial state, the final state and O stored or not; also on forced segments."""
    Bt, H, D = 2, 3, 96
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.bfloat16, 470 + N)
    u = synth.make_gate(Bt, H, N, D, torch.bfloat16, 470 + N)
    kv0 = torch.randn(Bt, H, D, D, generator=torch.Generator().manual_seed(N)) * 0.1
    decay = mixed_decay(H)
    o_ref, y_ref = orc.fwd_gated(q, k, v, u, decay, eps=1e-6, kv_in=kv0)
    _, kv_ref = orc.fwd_recurrent(q, k, v, decay, kv_in=kv0, return_state=True)
    with force_plan(segs=segs):
        _, y, kv = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6, kv_in=kv0.to(dev()),
                                          return_state=True, store_o=False)
    check("Y", y, y_ref, 1e-2)
    check("kv", kv, kv_ref, 1e-2)
    if segs == 0:
        # many chains: the library keeps the fused form with O stored too (192 chains and more)
        Bt2, H2 = 8, 24
        q, k, v = synth.make_qkv(Bt2, H2, N, D, torch.bfloat16, 480 + N)
        u = synth.make_gate(Bt2, H2, N, D, torch.bfloat16, 480 + N)
        decay = synth.decay_bench_rule(H2)
        o_ref, y_ref = orc.fwd_gated(q, k, v, u, decay, eps=1e-6)
        o, y = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6)
        check("O (192 chains)", o, o_ref, 1e-2)
        check("Y (192 chains)", y, y_ref, 1e-2)


def test_forward_gated_argument_errors():
    Bt, H, N, D = 1, 2, 64, 128
    q, k, v = gpu(*synth.make_qkv(Bt, H, N, D, torch.bfloat16, 3))
    u, = gpu(synth.make_gate(Bt, H, N, D, torch.bfloat16, 3))
    dd, = gpu(synth.decay_bench_rule(H))
    with pytest.raises(ltn.LtnError):
        ltn.ltn_attn_fwd_gated(q, k, v, u, dd, y_out=u)          # Y aliases the gate
    with pytest.raises(ltn.LtnError):
        ltn.ltn_attn_fwd_gated(q, k, v, u, dd, eps=float("nan"))


@pytest.mark.parametrize("D", [96, 128])
@pytest.mark.parametrize("N", [1, 64, 65, 193])
def test_bf16_many_chains_fused_with_o_stored(D, N):
    """192 chains with O stored run fused, the gate values of 96 and 128 features fetched within their block."""
    Bt, H = 24, 8
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.bfloat16, 480 + N)
    u = synth.make_gate(Bt, H, N, D, torch.bfloat16, 480 + N)
    decay = mixed_decay(H)
    o_ref, y_ref = orc.fwd_gated(q, k, v, u, decay, eps=1e-6)
    _, kv_ref = orc.fwd_recurrent(q, k, v, decay, return_state=True)
    o, y, kv = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6, return_state=True)
    check("O", o, o_ref, 1e-2)
    check("Y", y, y_ref, 1e-2)
    check("kv", kv, kv_ref, 1e-2)
    # the form without O fetches them a block ahead: the same values
    assert torch.equal(ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6, store_o=False)[1], y)
