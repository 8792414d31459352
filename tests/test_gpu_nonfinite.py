"""An infinity in one token of an fp32 call reaches what the definition lets it reach and nothing
else that a select or a zero row can keep it from: its own output row and the state come out
infinite (not NaN), and where the operand is masked by causality the other rows stay finite.
Lengths are ragged, so that the token sits next to the rows past the end of a short last block.
(An infinite value row meets zero scores of the earlier tokens of its own 16-token tile, and
0 x Inf is NaN there; those entries are left out.)

Finite entries are compared with the fp64 oracle at the fp32 bound of the parity suite."""
import numpy as np
import pytest
import torch

import paper_2307_14995_amd as ltn
from paper_2307_14995_amd import synth
from oracle import ltn_oracle as orc
from _helpers import TOL, force_plan, gpu

pytestmark = pytest.mark.gpu

F32 = torch.float32
H = 2
DECAY = torch.tensor([0.9, 1.0])
# (Dk, Dv, value columns per workgroup, N): every tile shape, tails of 1, 5 and 17 tokens
SHAPES = [(64, 64, 64, 37), (64, 64, 32, 65), (96, 96, 96, 69), (96, 96, 32, 81), (128, 128, 128, 69), (128, 128, 64, 33),
          (128, 128, 32, 49), (256, 256, 128, 21), (256, 256, 32, 33), (256, 128, 0, 37), (128, 64, 0, 69)]


def inputs(Dk, Dv, N):
    make = (lambda seed: synth.make_qkv(1, H, N, Dk, F32, seed)) if Dk == Dv else \
           (lambda seed: synth.make_qkv_dkdv(1, H, N, Dk, Dv, F32, seed))
    return (*make(500 + N), synth.make_do(1, H, N, Dv, F32, 500 + N))


def forward(Dk, Dv, dv, q, k, v):
    with force_plan(dv, 1):
        fn = ltn.ltn_attn_fwd if Dk == Dv else ltn.ltn_attn_fwd_dkdv
        o, kv = fn(*gpu(q, k, v, DECAY), return_state=True)
    return o.cpu().numpy(), kv.cpu().numpy()


def oracle(Dk, Dv, q, k, v):
    return (orc.fwd_recurrent if Dk == Dv else orc.fwd_recurrent_dkdv)(q, k, v, DECAY, return_state=True)


def close(got, ref):
    assert np.isfinite(got).all()
    return np.linalg.norm(got - ref) <= TOL[F32] * np.linalg.norm(ref)


@pytest.mark.parametrize("Dk,Dv,dv,N", SHAPES)
def test_infinite_key_in_the_last_token(Dk, Dv, dv, N):
    q, k, v, _ = inputs(Dk, Dv, N)
    o_ref, kv_ref = oracle(Dk, Dv, q, k, v)
    f = 5
    k[..., -1, f] = float("inf")
    o, kv = forward(Dk, Dv, dv, q, k, v)
    qn, vn = q.numpy(), v.numpy()
    assert (o[..., -1, :] == np.inf * np.sign(qn[..., -1, f, None] * vn[..., -1, :])).all()
    assert (kv[..., f, :] == np.inf * np.sign(vn[..., -1, :])).all()
    assert close(np.delete(kv, f, -2), np.delete(kv_ref, f, -2))


@pytest.mark.parametrize("Dk,Dv,dv,N", SHAPES)
def test_infinite_value_in_the_last_token(Dk, Dv, dv, N):
    q, k, v, _ = inputs(Dk, Dv, N)
    o_ref, kv_ref = oracle(Dk, Dv, q, k, v)
    j = 7
    v[..., -1, j] = float("inf")
    o, kv = forward(Dk, Dv, dv, q, k, v)
    score = (q.double() * k.double()).sum(-1).numpy()
    assert (o[..., -1, j] == np.inf * np.sign(score[..., -1])).all()
    assert close(np.delete(o, j, -1), np.delete(o_ref, j, -1))
    tile = (N - 1) // 16 * 16
    assert close(o[..., :tile, :], o_ref[..., :tile, :])
    assert (kv[..., j] == np.inf * np.sign(k.numpy()[..., -1, :])).all()
    assert close(np.delete(kv, j, -1), np.delete(kv_ref, j, -1))


@pytest.mark.parametrize("Dk,Dv,dv,N", SHAPES)
def test_infinite_query_in_the_first_token_of_the_reversed_pass(Dk, Dv, dv, N):
    """dV_0 = sum_t lambda^t (q_t . k_0) dO_t: the reversed pass meets token 0 last."""
    q, k, v, g = inputs(Dk, Dv, N)
    q[..., 0, 5] = float("inf")
    with force_plan(dv, 1):
        fn = ltn.ltn_attn_bwd if Dk == Dv else ltn.ltn_attn_bwd_dkdv
        dv_got = fn(*gpu(q, k, v, g, DECAY))[2].cpu().numpy()
    assert (dv_got[..., 0, :] == np.inf * np.sign(k.numpy()[..., 0, 5, None] * g.numpy()[..., 0, :])).all()


@pytest.mark.parametrize("Dk,Dv,dv,N", SHAPES)
def test_infinite_key_or_query_leaves_rows_masked_from_it_alone(Dk, Dv, dv, N):
    q, k, v, g = inputs(Dk, Dv, N)
    o_ref, _ = oracle(Dk, Dv, q, k, v)
    dv_ref = (orc.bwd_recurrent if Dk == Dv else orc.bwd_recurrent_dkdv)(q, k, v, g, DECAY)[2]
    t = 10                                 # inside a 16-token tile, neither first nor last
    ki, qi = k.clone(), q.clone()
    ki[..., t, 5] = float("inf")
    qi[..., t, 5] = float("inf")
    o, _ = forward(Dk, Dv, dv, q, ki, v)
    assert close(o[..., :t, :], o_ref[..., :t, :])
    assert (o[..., t, :] == np.inf * np.sign(q.numpy()[..., t, 5, None] * v.numpy()[..., t, :])).all()
    with force_plan(dv, 1):
        fn = ltn.ltn_attn_bwd if Dk == Dv else ltn.ltn_attn_bwd_dkdv
        dv_got = fn(*gpu(qi, k, v, g, DECAY))[2].cpu().numpy()
    assert close(dv_got[..., t + 1:, :], dv_ref[..., t + 1:, :])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("Dk,Dv", [(64, 64), (128, 64)])
def test_infinite_state_survives_segments_whose_decay_underflows(Dk, Dv, dtype):
    """0.5^256 is zero in fp32: cut or whole, a state entry that is infinite stays so."""
    N, H1 = 3 * 256 + 40, 2
    decay = torch.tensor([0.5, 0.0])
    q, k, v = (synth.make_qkv(1, H1, N, Dk, dtype, 77) if Dk == Dv else synth.make_qkv_dkdv(1, H1, N, Dk, Dv, dtype, 77))
    k[..., 3, 5] = float("inf")
    fn = ltn.ltn_attn_fwd if Dk == Dv else ltn.ltn_attn_fwd_dkdv
    got = {}
    for segs in (1, 3):
        with force_plan(0, segs):
            got[segs] = [x.float().cpu() for x in fn(*gpu(q, k, v, decay), return_state=True)]
    for whole, cut in zip(got[1], got[3]):
        assert torch.equal(whole[:, 0].isnan(), cut[:, 0].isnan())
        assert torch.equal(whole[:, 0].isinf(), cut[:, 0].isinf())
        bad = ~whole[:, 0].isfinite()
        assert bad.any() and torch.equal(whole[:, 0][bad].sign().nan_to_num(), cut[:, 0][bad].sign().nan_to_num())
    # lambda = 0: the state of the last token alone, which is finite; 0 x Inf in either form before it
    assert torch.equal(got[1][1][:, 1].isnan(), got[3][1][:, 1].isnan())
