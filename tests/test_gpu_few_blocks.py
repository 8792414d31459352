"""Chains of one to six 64-token blocks, fewer than the tile ring has stages and a few more, in every
slice width: the ring's start, what each wait counts there, and the states that come in before the
first block.  Against the fp64 oracle with the parity suite's tolerances."""
import pytest
import torch

import paper_2307_14995_amd as ltn
from paper_2307_14995_amd import synth
from oracle import ltn_oracle as orc
from _helpers import TOL, check, force_dv, gpu, mixed_decay

pytestmark = pytest.mark.gpu
BF = torch.bfloat16
LENGTHS = [64, 100, 128, 192, 200, 256, 300, 384]
SLICES = [(64, 64), (64, 32), (96, 96), (96, 32), (128, 128), (128, 64), (128, 32), (256, 64), (256, 32)]


@pytest.mark.parametrize("D,dv", SLICES)
@pytest.mark.parametrize("N", LENGTHS)
def test_forward_and_gradients(D, dv, N):
    q, k, v = synth.make_qkv(1, 4, N, D, BF, 700 + N)
    g = synth.make_do(1, 4, N, D, BF, 700 + N)
    decay = mixed_decay(4)
    kv0 = torch.randn(1, 4, D, D, generator=torch.Generator().manual_seed(N)) / D
    o_ref, kv_ref = orc.fwd_recurrent(q, k, v, decay, kv_in=kv0, return_state=True)
    with force_dv(dv):
        o, kv = ltn.ltn_attn_fwd(*gpu(q, k, v, decay), kv_in=kv0.cuda(), return_state=True)
        grads = ltn.ltn_attn_bwd(*gpu(q, k, v, g, decay))
    check("O", o, o_ref, TOL[BF])
    check("kv", kv, kv_ref, TOL[BF])
    for n, x, r in zip(("dQ", "dK", "dV"), grads, orc.bwd_recurrent(q, k, v, g, decay)):
        check(n, x, r, TOL[BF])


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("N", LENGTHS)
@pytest.mark.parametrize("store_o", [False, True])
def test_gated_forward(D, N, store_o):
    # 200 chains: one launch, also where the output is stored
    q, k, v = synth.make_qkv(50, 4, N, D, BF, 720 + N)
    u = synth.make_gate(50, 4, N, D, BF, 720 + N)
    decay = mixed_decay(4)
    o_ref, y_ref = orc.fwd_gated(q, k, v, u, decay, eps=1e-6)
    o, y = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6, store_o=store_o)
    check("Y", y, y_ref, TOL[BF])
    if store_o:
        check("O", o, o_ref, TOL[BF])


@pytest.mark.parametrize("Dk", [256, 128])
@pytest.mark.parametrize("N", LENGTHS)
def test_unequal_widths(Dk, N):
    q, k, v = synth.make_qkv_dkdv(1, 4, N, Dk, Dk // 2, BF, 740 + N)
    g = synth.make_do(1, 4, N, Dk // 2, BF, 740 + N)
    decay = mixed_decay(4)
    check("O", ltn.ltn_attn_fwd_dkdv(*gpu(q, k, v, decay)), orc.fwd_recurrent_dkdv(q, k, v, decay), TOL[BF])
    for n, x, r in zip(("dQ", "dK", "dV"), ltn.ltn_attn_bwd_dkdv(*gpu(q, k, v, g, decay)),
                       orc.bwd_recurrent_dkdv(q, k, v, g, decay)):
        check(n, x, r, TOL[BF])


@pytest.mark.parametrize("chains,store_o", [(127, False), (128, False), (191, True), (192, True)])
@pytest.mark.parametrize("N", [65, 256, 257, 449])
def test_gate_values_on_both_sides_of_the_line(chains, store_o, N):
    # heads of 64 features: gate values fetched one block ahead, and two from so many chains and more than four blocks on
    q, k, v = synth.make_qkv(1, chains, N, 64, BF, 760 + N)
    u = synth.make_gate(1, chains, N, 64, BF, 760 + N)
    decay = mixed_decay(chains)
    kv0 = torch.randn(1, chains, 64, 64, generator=torch.Generator().manual_seed(N)) / 64
    o_ref, kv_ref = orc.fwd_recurrent(q, k, v, decay, kv_in=kv0, return_state=True)
    y_ref = orc.gate_fwd(o_ref, u, eps=1e-6)
    _, y, kv = ltn.ltn_attn_fwd_gated(*gpu(q, k, v, u, decay), eps=1e-6, kv_in=kv0.cuda(), return_state=True,
                                      store_o=store_o)
    check("Y", y, y_ref, TOL[BF])
    check("kv", kv, kv_ref, TOL[BF])
