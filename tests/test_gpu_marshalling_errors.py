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
IN_PYTHON = ("ltn_gate_fwd", "ltn_attn_fwd_tiled", "ltn_attn_bwd_tiled", "ltn_attn_fwd_static")


class StandIn:
    """The library, with every launching entry point replaced; `calls` holds the names as they are called."""
    def __init__(self, lib, status):
        self._lib, self.calls = lib, []
        for name in LAUNCHING + IN_PYTHON:
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


def with_outputs(bad):
    """Calls with one output of the caller's each, by entry point and argument: `bad` makes the output from one
    that would do."""
    q, k, v = synth.make_qkv(Bt, H, N, D, torch.bfloat16, 3)
    q, k, v, decay, theta = gpu(q, k, v, synth.decay_bench_rule(H), synth.make_theta(H, D, 3))
    w = torch.cat((q, k), -1)
    kv, kvw = torch.zeros(Bt, H, D, D, device="cuda"), torch.zeros(Bt, H, 2 * D, D, device="cuda")
    q1 = q[:, :, 0].contiguous()
    o, o1, s, sw = (bad(torch.empty_like(t)) for t in (q, q1, kv, kvw))
    a, b = torch.empty_like(q), torch.empty_like(q)
    return {
        "fwd out": lambda: ltn.ltn_attn_fwd(q, k, v, decay, out=o),
        "fwd kv_out": lambda: ltn.ltn_attn_fwd(q, k, v, decay, kv_out=s),
        "gated out": lambda: ltn.ltn_attn_fwd_gated(q, k, v, q, decay, out=o),
        "gated y_out": lambda: ltn.ltn_attn_fwd_gated(q, k, v, q, decay, y_out=o),
        "gated y_out alone": lambda: ltn.ltn_attn_fwd_gated(q, k, v, q, decay, y_out=o, store_o=False),
        "gated kv_out": lambda: ltn.ltn_attn_fwd_gated(q, k, v, q, decay, kv_out=s),
        "gate": lambda: ltn.ltn_gate_fwd(q, k, out=o),
        "gate bwd dx": lambda: ltn.ltn_gate_bwd(q, k, v, out=(o, a)),
        "gate bwd du": lambda: ltn.ltn_gate_bwd(q, k, v, out=(a, o)),
        "bwd dq": lambda: ltn.ltn_attn_bwd(q, k, v, q, decay, out=(o, a, b)),
        "bwd dv": lambda: ltn.ltn_attn_bwd(q, k, v, q, decay, out=(a, b, o)),
        "step": lambda: ltn.ltn_attn_decode_step(q1, q1, q1, kv, decay, out=o1),
        "steps": lambda: ltn.ltn_attn_decode_steps(q, k, v, kv, decay, out=o),
        "tiled": lambda: ltn.ltn_attn_fwd_tiled(q, k, v, decay, out=o),
        "tiled bwd": lambda: ltn.ltn_attn_bwd_tiled(q, k, v, q, decay, out=(a, o, b)),
        "dkdv out": lambda: ltn.ltn_attn_fwd_dkdv(w, w, v, decay, out=o),
        "dkdv kv_out": lambda: ltn.ltn_attn_fwd_dkdv(w, w, v, decay, kv_out=sw),
        "steps dkdv": lambda: ltn.ltn_attn_decode_steps_dkdv(w, w, v, kvw, decay, out=o),
        "swish": lambda: ltn.ltn_prologue_fwd(q, out=o),
        "static": lambda: ltn.ltn_attn_fwd_static(q, k, v, decay, o),
        "static kv_out": lambda: ltn.ltn_attn_fwd_static(q, k, v, decay, a, kv_out=s),
    }


BAD = {
    "short": lambda t: t.flatten()[:-1],
    "another type": lambda t: t.to(torch.float32 if t.dtype == torch.bfloat16 else torch.bfloat16),
    "strided": lambda t: torch.cat((t, t), -1)[..., ::2],
    "on the host": lambda t: t.cpu(),
}


@pytest.mark.parametrize("bad", BAD)
@pytest.mark.parametrize("through", ["both", "python"])
def test_an_output_that_the_call_does_not_fit_is_refused(stand_in, monkeypatch, bad, through):
    lib = stand_in(0)
    if through == "python":
        monkeypatch.setattr(binding, "_native", type("Declines", (), {"__getattr__": lambda self, n: lambda *args: None})())
    for name, call in with_outputs(BAD[bad]).items():
        with pytest.raises(ValueError):
            call()
            pytest.fail(f"{name}: an output {bad} was accepted", pytrace=False)
    assert lib.calls == []


def test_a_longer_output_or_another_shape_is_taken(stand_in):
    # as many elements as the call writes, or more: the caller's own affair
    lib = stand_in(0)
    exact = ("swish", "static", "static kv_out")           # these have always asked for the shape
    for more in (lambda t: t.flatten(), lambda t: torch.cat((t, t)).flatten()):
        fns = with_outputs(more)
        for name in fns:
            if name not in exact:
                fns[name]()
    assert len(lib.calls) == 2 * (len(fns) - len(exact))
