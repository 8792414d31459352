"""What the native marshalling does with calls that fail.  The library's entry points are replaced by
stand-ins that count their calls, launch nothing and return a status, so no GPU error is needed."""
import ctypes

import pytest
import torch

import paper_2307_14995_amd as ltn
from paper_2307_14995_amd import binding, synth
from _helpers import gpu

pytestmark = pytest.mark.gpu

Bt, H, N, D = 1, 2, 70, 64
LAUNCHING = ("ltn_attn_fwd", "ltn_attn_fwd_gated", "ltn_attn_bwd", "ltn_gate_bwd", "ltn_attn_decode_step",
             "ltn_attn_decode_steps", "ltn_attn_fwd_dkdv", "ltn_attn_bwd_dkdv", "ltn_attn_decode_steps_dkdv",
             "ltn_prologue_fwd", "ltn_prologue_bwd")


class StandIn:
    """The library, with every launching entry point replaced; `calls` holds the names as they are called."""
    def __init__(self, lib, status):
        self._lib, self.calls = lib, []
        for name in LAUNCHING:
            def stub(*args, name=name):
                self.calls.append(name)
                return status
            setattr(self, name, ctypes.CFUNCTYPE(ctypes.c_int, *getattr(lib, name).argtypes)(stub))

    def __getattr__(self, name):
        return getattr(self._lib, name)


@pytest.fixture
def stand_in(monkeypatch):
    real = binding.load_library()

    def put(status):
        lib = StandIn(real, status)
        monkeypatch.setattr(binding, "_lib", lib)
        binding._bind_native(lib)
        return lib

    yield put
    binding._bind_native(real)


def entries(refuse=False):
    """Every entry point that is marshalled natively, as a call of plain arguments; `refuse`: with one
    input whose storage refuses access."""
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.bfloat16, 3)
    q, k, v, decay, theta = gpu(q, k, v, synth.decay_bench_rule(H), synth.make_theta(H, D, 3))
    w = torch.cat((q, k), -1)
    kv, kvw = torch.zeros(Bt, H, D, D, device="cuda"), torch.zeros(Bt, H, 2 * D, D, device="cuda")
    q1 = q[:, :, 0].contiguous()
    for t in (q, w, q1) if refuse else ():
        torch._C._set_throw_on_mutable_data_ptr(t)
    return {
        "ltn_attn_fwd": lambda: ltn.ltn_attn_fwd(q, k, v, decay, kv_in=kv, kv_out=kv),
        "ltn_attn_fwd_gated": lambda: ltn.ltn_attn_fwd_gated(q, k, v, q, decay, kv_in=kv, kv_out=kv),
        "ltn_attn_bwd": lambda: ltn.ltn_attn_bwd(q, k, v, q, decay),
        "ltn_gate_bwd": lambda: ltn.ltn_gate_bwd(q, k, v),
        "ltn_attn_decode_step": lambda: ltn.ltn_attn_decode_step(q1, q1, q1, kv, decay),
        "ltn_attn_decode_steps": lambda: ltn.ltn_attn_decode_steps(q, k, v, kv, decay),
        "ltn_attn_fwd_dkdv": lambda: ltn.ltn_attn_fwd_dkdv(w, w, v, decay, kv_in=kvw, kv_out=kvw),
        "ltn_attn_bwd_dkdv": lambda: ltn.ltn_attn_bwd_dkdv(w, w, v, v, decay),
        "ltn_attn_decode_steps_dkdv": lambda: ltn.ltn_attn_decode_steps_dkdv(w, w, v, kvw, decay),
        "ltn_prologue_fwd": lambda: ltn.ltn_prologue_fwd(q, theta),
        "ltn_prologue_bwd": lambda: ltn.ltn_prologue_bwd(q, w, theta),
    }


@pytest.mark.parametrize("name", LAUNCHING)
@pytest.mark.parametrize("status", [6, 77])
def test_a_failed_launch_is_reported_and_not_repeated(stand_in, name, status):
    # a status that is not found before the first launch: work may be in flight, states already advanced
    call = entries()[name]
    lib = stand_in(status)
    with pytest.raises(ltn.LtnError, match=name + ":") as e:
        call()
    assert e.value.code == status
    assert len(lib.calls) == 1


@pytest.mark.parametrize("name", LAUNCHING)
def test_a_refused_argument_raises(stand_in, name):
    call = entries()[name]
    stand_in(3)
    with pytest.raises(ltn.LtnError, match=name + ":") as e:
        call()
    assert e.value.code == 3


@pytest.mark.parametrize("name", LAUNCHING)
def test_an_input_without_an_address_raises(name):
    # (found while the interpreter is released: it has to be held again before the error is raised)
    with pytest.raises(RuntimeError, match="data pointer"):
        entries(refuse=True)[name]()
    entries()[name]()
