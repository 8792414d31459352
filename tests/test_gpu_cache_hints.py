"""Calls large enough for cache hints (non-temporal loads, outputs and states stored through or past the caches): the
same bits as the two halves of the batch, which are below the sizes where hints begin."""
import pytest
import torch

import paper_2307_14995_amd as ltn
from _helpers import force_plan, mixed_decay

pytestmark = pytest.mark.gpu


def rand(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)


def inputs(H, N, D, n):
    g = torch.Generator(device="cuda").manual_seed(N)
    return [rand(g, 2, H, N, D) for _ in range(n)], mixed_decay(H).cuda()


def halves(call, tensors, dv, segs):
    """call on each half of the batch (its only dimension but chains), under a forced plan"""
    with force_plan(dv=dv, segs=segs):
        parts = [call(*(t[i:i + 1].contiguous() for t in tensors)) for i in range(2)]
    return [torch.cat(p) for p in zip(*parts)]


# (D, H, N, dv, segs) of half the chains: segments of full width
@pytest.mark.parametrize("D,H,N,dv,segs", [(128, 16, 13000, 128, 8), (128, 4, 51300, 128, 8)])
def test_forward(D, H, N, dv, segs):
    t, decay = inputs(H, N, D, 3)
    with force_plan(dv=dv, segs=segs):
        o, kv = ltn.ltn_attn_fwd(*t, decay, return_state=True)
    want = halves(lambda *x: ltn.ltn_attn_fwd(*x, decay, return_state=True), t, dv, segs)
    assert torch.equal(o, want[0]) and torch.equal(kv, want[1])


# without o (with it there are no hints); 64 features with up to four blocks, whose kernel is another, and in segments too
@pytest.mark.parametrize("D,H,N,segs", [(128, 192, 137, 1), (96, 192, 190, 1), (64, 192, 300, 1), (64, 192, 1217, 1), (64, 210, 250, 1),
                                        (128, 200, 705, 1), (96, 200, 769, 1), (128, 16, 5000, 8), (64, 16, 9900, 8)])
def test_gated_forward(D, H, N, segs):
    t, decay = inputs(H, N, D, 4)

    def call(*x):
        return ltn.ltn_attn_fwd_gated(*x, decay, eps=1e-6, return_state=True, store_o=False)[1:]

    with force_plan(segs=segs if segs > 1 else 0):
        got = call(*t)
    assert all(torch.equal(a, b) for a, b in zip(got, halves(call, t, 0, segs)))


# both by themselves (dQ's chains may run in two parts) and in whole chains
@pytest.mark.parametrize("D,H,N", [(128, 64, 1921), (96, 86, 1921), (64, 154, 1921), (128, 100, 1250)])
def test_backward(D, H, N):
    t, decay = inputs(H, N, D, 4)
    want = halves(lambda *x: ltn.ltn_attn_bwd(*x, decay), t, D, 1)
    assert all(torch.equal(a, b) for a, b in zip(ltn.ltn_attn_bwd(*t, decay), want))
    with force_plan(segs=1):
        assert all(torch.equal(a, b) for a, b in zip(ltn.ltn_attn_bwd(*t, decay), want))


# in segments of full width: inputs of 241 and 289 MiB
@pytest.mark.parametrize("D,H,N", [(128, 8, 15400), (64, 8, 37000)])
def test_backward_in_segments(D, H, N):
    t, decay = inputs(H, N, D, 4)
    with force_plan(dv=D, segs=5):
        assert ltn.ltn_attn_query_plan(2, H, N, D, torch.bfloat16, 1) == (D, 5)
        got = ltn.ltn_attn_bwd(*t, decay)
    want = halves(lambda *x: ltn.ltn_attn_bwd(*x, decay), t, D, 5)
    assert all(torch.equal(a, b) for a, b in zip(got, want))


# states of the size that is written through, and the halves, which are not
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("Dk,Dv,chains,steps", [(128, 128, 640, 1), (128, 128, 1152, 1), (128, 128, 1152, 3), (256, 256, 96, 2), (64, 64, 1536, 1),
                                                (96, 96, 1140, 2), (128, 64, 1280, 1), (256, 128, 192, 1)])
def test_decode(Dk, Dv, chains, steps, dtype):
    g = torch.Generator(device="cuda").manual_seed(chains)
    q, k, v = (torch.randn(2, chains // 2, steps, D, generator=g, device="cuda").to(dtype) for D in (Dk, Dk, Dv))
    kv = torch.randn(2, chains // 2, Dk, Dv, generator=g, device="cuda")
    decay = mixed_decay(chains // 2).cuda()
    call = ltn.ltn_attn_decode_steps if Dk == Dv else ltn.ltn_attn_decode_steps_dkdv
    parts = [kv[i:i + 1].clone() for i in range(2)]
    want = [call(*(t[i:i + 1].contiguous() for t in (q, k, v)), parts[i], decay) for i in range(2)]
    o = call(q, k, v, kv, decay)
    assert torch.equal(o, torch.cat(want)) and torch.equal(kv, torch.cat(parts))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D", [128, 96, 64, 256])
@pytest.mark.parametrize("mib", [24, 64])              # of a tensor: where hints begin, and the forward's for y
def test_gate(D, mib, dtype):
    g = torch.Generator(device="cuda").manual_seed(D)
    rows = 2 * -(-(mib << 20) // (2 * D * dtype.itemsize))
    x, u, dy = (torch.randn(1, 2, rows // 2, D, generator=g, device="cuda").to(dtype) for _ in range(3))
    got = [ltn.ltn_gate_fwd(x, u, eps=1e-6), *ltn.ltn_gate_bwd(x, u, dy, eps=1e-6)]
    parts = [[t[:, i:i + 1].contiguous() for t in (x, u, dy)] for i in range(2)]
    want = [[ltn.ltn_gate_fwd(p[0], p[1], eps=1e-6), *ltn.ltn_gate_bwd(*p, eps=1e-6)] for p in parts]
    for a, *b in zip(got, *want):
        assert torch.equal(a, torch.cat(b, 1))


# batch entries whose loads are issued one, two and four at a time, with remainders, below and above the line for hints
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D,Bt,H,N", [(128, 2, 16, 2049), (128, 6, 4, 2801), (128, 18, 2, 2000), (64, 18, 8, 1000),
                                      (64, 10, 3, 70), (64, 5, 3, 70), (128, 1, 3, 65)])
def test_input_side(D, Bt, H, N, dtype):
    g = torch.Generator(device="cuda").manual_seed(N)
    x = torch.randn(Bt, H, N, D, generator=g, device="cuda").to(dtype)
    dy = torch.randn(Bt, H, N, 2 * D, generator=g, device="cuda").to(dtype)
    theta = torch.rand(H, D, generator=g, device="cuda")
    y = ltn.ltn_prologue_fwd(x, theta, pos0=5)
    dx, dth = ltn.ltn_prologue_bwd(x, dy, theta, pos0=5)
    one = [(ltn.ltn_prologue_fwd(x[b:b + 1].contiguous(), theta, pos0=5),
            *ltn.ltn_prologue_bwd(x[b:b + 1].contiguous(), dy[b:b + 1].contiguous(), theta, pos0=5)) for b in range(Bt)]
    assert torch.equal(y, torch.cat([o[0] for o in one])) and torch.equal(dx, torch.cat([o[1] for o in one]))
    # sums over the batch in another order: at most Bt kTok / TY = 288 fp32 terms a thread
    ref = torch.stack([o[2] for o in one]).double().sum(0)
    assert (dth.double() - ref).norm() <= 288 * 2.0 ** -24 * torch.stack([o[2] for o in one]).double().abs().sum(0).norm()
