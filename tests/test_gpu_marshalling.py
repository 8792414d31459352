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


class Recorder:
    """The native module, keeping for each entry whether it did the call itself."""
    def __init__(self, module):
        self.module, self.did = module, {}

    def __getattr__(self, name):
        def call(*args):
            r = getattr(self.module, name)(*args)
            self.did.setdefault(name, []).append(r is not None)
            return r
        return call


#: entries of the native module, and how many of calls() go through each
ENTRIES = {"fwd": 2, "fwd_gated": 2, "bwd": 1, "gate_bwd": 1, "decode_step": 1, "decode_steps": 1, "fwd_dkdv": 1,
           "bwd_dkdv": 1, "decode_steps_dkdv": 1, "prologue_fwd": 2, "prologue_bwd": 2}


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
    recorder = Recorder(binding._fast())
    monkeypatch.setattr(binding, "_native", recorder)
    native = {n: flat(f()) for n, f in fns.items()}
    assert recorder.did == {n: [True] * c for n, c in ENTRIES.items()}         # none of them by way of Python
    monkeypatch.setattr(binding, "_native", Refuses())
    for n, f in fns.items():
        python = flat(f())
        assert len(native[n]) == len(python), n
        for a, b in zip(native[n], python):
            assert (a is None) == (b is None), n
            assert a is None or (a.dtype == b.dtype and torch.equal(a, b)), n


def test_callers_outputs_come_back(monkeypatch):
    recorder = Recorder(binding._fast())
    monkeypatch.setattr(binding, "_native", recorder)
    q, k, v, u, _, decay, _ = inputs(torch.bfloat16)
    o, y, kv = torch.empty_like(q), torch.empty_like(q), torch.empty(Bt, H, D, D, device="cuda")
    r = ltn.ltn_attn_fwd(q, k, v, decay, out=o, kv_out=kv)
    assert r[0] is o and r[1] is kv
    r = ltn.ltn_attn_fwd_gated(q, k, v, u, decay, out=o, y_out=y, kv_out=kv)
    assert r[0] is o and r[1] is y and r[2] is kv
    q1 = q[:, :, 0].contiguous()
    o1 = torch.empty_like(q1)
    assert ltn.ltn_attn_decode_step(q1, q1, q1, kv, decay, out=o1) is o1
    assert recorder.did == {"fwd": [True], "fwd_gated": [True], "decode_step": [True]}


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


def native_arguments(dtype):
    """The arguments that binding.py hands to each entry of the native module."""
    q, k, v, u, g, decay, theta = inputs(dtype)
    w = torch.cat((q, k), -1)
    kv, kvw = torch.zeros(Bt, H, D, D, device="cuda"), torch.zeros(Bt, H, 2 * D, D, device="cuda")
    q1, k1, v1 = (x[:, :, 3].contiguous() for x in (q, k, v))
    return {
        "fwd": [q, k, v, decay, kv, True, 0, None, None],
        "fwd_gated": [q, k, v, u, decay, 0.0, kv, True, True, 0, None, None, None],
        "bwd": [q, k, v, g, decay, 0],
        "gate_bwd": [q, u, g, 0.0],
        "decode_step": [q1, k1, v1, kv, decay, None],
        "decode_steps": [q, k, v, kv, decay, None],
        "fwd_dkdv": [w, w, v, decay, kvw, True, 0, None, None],
        "bwd_dkdv": [w, w, v, g, decay, 0],
        "decode_steps_dkdv": [w, w, v, kvw, decay, None],
        "prologue_fwd": [q, theta, True, 0, None],
        "prologue_bwd": [q, w, theta, True, 0, True],
    }


@pytest.mark.parametrize("entry", ENTRIES)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_every_entry_refuses_each_wrong_argument(entry, dtype):
    # one argument at a time, in the place of one that is taken: left to Python, nothing is launched
    native, args = getattr(binding._fast(), entry), native_arguments(dtype)[entry]
    assert native(*args) is not None
    for i, a in enumerate(args):
        if isinstance(a, torch.Tensor):
            wrong = [a.cpu(), a.half(), a[..., :-1], a[..., :-1].contiguous(), torch.cat((a, a), -1)[..., ::2], 1, "x"]
        elif a is None:
            wrong = [1, "x", torch.empty(1, device="cuda"), torch.empty(Bt, H, N, 2 * D, dtype=torch.half, device="cuda")]
        elif isinstance(a, bool):
            wrong = [1, None, "x"]
        elif isinstance(a, float):
            wrong = [None, "x", torch.zeros(1)]
        else:
            wrong = [None, "x", 1.0, 1 << 70]
        for w in wrong:
            assert native(*args[:i], w, *args[i + 1:]) is None, (i, w)
    assert native(*args[:-1]) is None and native(*args, None) is None
