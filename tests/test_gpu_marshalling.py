"""The native marshalling against the Python path behind it: the same bits from every entry point, the
caller's own tensors handed back, and anything that is not the plain case left to Python."""
import pytest
import torch

import paper_2307_14995_amd as ltn
from paper_2307_14995_amd import binding, synth
from _helpers import gpu

pytestmark = pytest.mark.gpu

Bt, H, N, D = 2, 3, 70, 64


class Refuses:
    """In the place of the native module: every call goes on in Python."""
    def __getattr__(self, name):
        return lambda *args: None


def inputs(dtype):
    q, k, v = synth.make_qkv(Bt, H, N, D, dtype, 5)
    u, g = synth.make_gate(Bt, H, N, D, dtype, 5), synth.make_do(Bt, H, N, D, dtype, 5)
    return gpu(q, k, v, u, g, synth.decay_bench_rule(H), synth.make_theta(H, D, 5))


def flat(x):
    return [y for z in x for y in flat(z)] if isinstance(x, tuple) else [x]


def calls(q, k, v, u, g, decay, theta):
    kv, kvw = torch.randn(Bt, H, D, D, device="cuda"), torch.randn(Bt, H, 2 * D, D, device="cuda")
    w = ltn.ltn_prologue_fwd(q, theta)
    one = [x[:, :, 3].contiguous() for x in (q, k, v)]
    some = [x[:, :, :3].contiguous() for x in (q, k, v, w)]

    def step(fn, *args):
        state = (kvw if "dkdv" in fn.__name__ else kv).clone()
        return lambda: (fn(*args, state.copy_(kvw if "dkdv" in fn.__name__ else kv), decay), state.clone())

    return {
        "fwd": lambda: ltn.ltn_attn_fwd(q, k, v, decay),
        "fwd state": lambda: ltn.ltn_attn_fwd(q, k, v, decay, kv_in=kv, return_state=True, block=64 if q.dtype == torch.bfloat16 else 0),
        "gated": lambda: ltn.ltn_attn_fwd_gated(q, k, v, u, decay, eps=1e-6),
        "gated no o": lambda: ltn.ltn_attn_fwd_gated(q, k, v, u, decay, eps=0, kv_in=kv, return_state=True, store_o=False),
        "bwd": lambda: ltn.ltn_attn_bwd(q, k, v, g, decay),
        "gate bwd": lambda: ltn.ltn_gate_bwd(q, u, g, eps=1e-6),
        "step": step(ltn.ltn_attn_decode_step, *one),
        "steps": step(ltn.ltn_attn_decode_steps, *some[:3]),
        "fwd dkdv": lambda: ltn.ltn_attn_fwd_dkdv(w, w, v, decay, kv_in=kvw, return_state=True),
        "bwd dkdv": lambda: ltn.ltn_attn_bwd_dkdv(w, w, v, g, decay),
        "steps dkdv": step(ltn.ltn_attn_decode_steps_dkdv, some[3], some[3], some[2]),
        "prologue": lambda: ltn.ltn_prologue_fwd(q, theta, pos0=7),
        "swish": lambda: ltn.ltn_prologue_fwd(q),
        "prologue bwd": lambda: ltn.ltn_prologue_bwd(q, w, theta),
        "swish bwd": lambda: ltn.ltn_prologue_bwd(q, g),
    }


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_same_bits_as_the_python_path(dtype, monkeypatch):
    fns = calls(*inputs(dtype))
    native = {n: flat(f()) for n, f in fns.items()}
    monkeypatch.setattr(binding, "_native", Refuses())
    for n, f in fns.items():
        python = flat(f())
        assert len(native[n]) == len(python), n
        for a, b in zip(native[n], python):
            assert (a is None) == (b is None), n
            assert a is None or (a.dtype == b.dtype and torch.equal(a, b)), n


def test_callers_outputs_come_back():
    q, k, v, u, _, decay, _ = inputs(torch.bfloat16)
    o, y, kv = torch.empty_like(q), torch.empty_like(q), torch.empty(Bt, H, D, D, device="cuda")
    r = ltn.ltn_attn_fwd(q, k, v, decay, out=o, kv_out=kv)
    assert r[0] is o and r[1] is kv
    r = ltn.ltn_attn_fwd_gated(q, k, v, u, decay, out=o, y_out=y, kv_out=kv)
    assert r[0] is o and r[1] is y and r[2] is kv
    q1 = q[:, :, 0].contiguous()
    o1 = torch.empty_like(q1)
    assert ltn.ltn_attn_decode_step(q1, q1, q1, kv, decay, out=o1) is o1


def test_what_is_not_plain_is_left_to_python():
    q, k, v, _, _, decay, _ = inputs(torch.bfloat16)
    fwd = binding._fast().fwd

    def fast(q=q, k=k, v=v, decay=decay, kv_in=None, want=False, block=0, out=None, kv_out=None):
        return fwd(q, k, v, decay, kv_in, want, block, out, kv_out)

    assert torch.equal(fast(), ltn.ltn_attn_fwd(q, k, v, decay))
    assert fast(q=torch.nn.Parameter(q)) is not None

    class Sub(torch.Tensor):
        pass

    for bad in (dict(q=q.cpu()), dict(q=q.as_subclass(Sub)), dict(k=k[:, :, 1:]), dict(v=v.float()), dict(decay=decay[:-1]),
                dict(decay=decay.double()), dict(q=q.transpose(1, 2)), dict(block=7), dict(block=1 << 40), dict(want=1),
                dict(kv_in=q), dict(q=None), dict(q=q.half(), k=k.half(), v=v.half()), dict(out=q)):
        assert fast(**bad) is None
    assert fwd(q, k, v) is None
    with pytest.raises(ltn.LtnError):      # an output over an input: the library's own refusal
        ltn.ltn_attn_fwd(q, k, v, decay, out=q)
    with pytest.raises(ValueError):
        ltn.ltn_attn_fwd(q, k, v, decay[:-1])
    assert torch.equal(ltn.ltn_attn_fwd(q.as_subclass(Sub), k, v, decay), ltn.ltn_attn_fwd(q, k, v, decay))
    with torch.inference_mode(), torch.device("cpu"):              # an active function mode
        assert fast() is None and ltn.ltn_attn_fwd(q, k, v, decay).is_cuda


def test_captured_call_replays():
    q, k, v, _, g, decay, _ = inputs(torch.bfloat16)
    ref = ltn.ltn_attn_bwd(q, k, v, g, decay)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        side = ltn.ltn_attn_bwd(q, k, v, g, decay)                 # the current stream, whichever it is
    s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = ltn.ltn_attn_bwd(q, k, v, g, decay)
    for _ in range(3):
        for x in got:
            x.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) and torch.equal(a, c) for a, b, c in zip(ref, got, side))
