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
