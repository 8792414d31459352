"""Decode by 32-column slices and by whole states: both sides of the line between them, every width and
tensor type, one token and several, against the fp64 oracle; and a call of several tokens has the bits
of as many calls of one on either side.  Bounds: the parity suite's."""
import pytest
import torch

import paper_2307_14995_amd as ltn
from paper_2307_14995_amd import synth
from oracle import ltn_oracle as orc
from _helpers import TOL, check, gpu, mixed_decay

pytestmark = pytest.mark.gpu

# (Dk, Dv, last number of chains that is split)
LINES = [(64, 64, 0), (96, 96, 512), (128, 128, 384), (128, 64, 512), (256, 128, 2048), (256, 256, 1024)]


def run(Dk, Dv, Bt, H, S, dtype):
    q, k, v = (synth.make_qkv(Bt, H, S, Dk, dtype, 31) if Dk == Dv else synth.make_qkv_dkdv(Bt, H, S, Dk, Dv, dtype, 31))
    decay = mixed_decay(H)
    kv = torch.randn(Bt, H, Dk, Dv, generator=torch.Generator().manual_seed(Dk)) / Dk
    fn = ltn.ltn_attn_decode_steps if Dk == Dv else ltn.ltn_attn_decode_steps_dkdv
    qd, kd, vd, dd = gpu(q, k, v, decay)
    state = kv.cuda()
    o = fn(qd, kd, vd, state, dd)
    one = kv.cuda()
    rows = [fn(*(x[:, :, t:t + 1].contiguous() for x in (qd, kd, vd)), one, dd) for t in range(S)]
    assert torch.equal(torch.cat(rows, 2), o) and torch.equal(one, state)
    fwd = orc.fwd_recurrent if Dk == Dv else orc.fwd_recurrent_dkdv
    o_ref, kv_ref = fwd(q, k, v, decay, kv_in=kv, return_state=True)
    check("O", o, o_ref, TOL[dtype], per_slice=False)
    check("kv", state, kv_ref, TOL[torch.float32])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("Dk,Dv,last", LINES)
@pytest.mark.parametrize("chains,S", [(1, 3), (7, 1)])
def test_few_chains(Dk, Dv, last, chains, S, dtype):
    run(Dk, Dv, 1, chains, S, dtype)


@pytest.mark.parametrize("Dk,Dv,last", LINES[1:])
@pytest.mark.parametrize("past", [0, 1])
def test_both_sides_of_the_line(Dk, Dv, last, past):
    run(Dk, Dv, last + past, 1, 2, torch.bfloat16)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("Dk,Dv,last", LINES[1:])
@pytest.mark.parametrize("S", [1, 3])
def test_a_sequence_does_not_depend_on_its_batch(Dk, Dv, last, S, dtype):
    # the same chains in a call of whole states, of slices, and of few: the same bits
    q, k, v = (synth.make_qkv(last + 1, 1, S, Dk, dtype, 33) if Dk == Dv else
               synth.make_qkv_dkdv(last + 1, 1, S, Dk, Dv, dtype, 33))
    fn = ltn.ltn_attn_decode_steps if Dk == Dv else ltn.ltn_attn_decode_steps_dkdv
    q, k, v, decay = gpu(q, k, v, torch.tensor([0.97]))
    kv = torch.randn(last + 1, 1, Dk, Dv, generator=torch.Generator("cuda").manual_seed(Dk), device="cuda") / Dk
    got = []
    for n in (last + 1, last, 3):
        state = kv[:n].clone()
        got.append((fn(q[:n], k[:n], v[:n], state, decay), state))
    for n in (last, 3):
        o, state = got.pop()
        assert torch.equal(o, got[0][0][:o.shape[0]]) and torch.equal(state, got[0][1][:o.shape[0]])
