"""The work that users of this library have it do, as timed cases.

Five kinds of pass, each through the public entry points of the Python binding:

  train        one attention layer's training step: forward, then dQ, dK, dV
  mixer        the whole token mixer's training step: gated forward with the attention output
               stored, derivative of the gate, attention gradients
  prefill      a prompt, or the next chunk of one, in inference: gated forward without the
               attention output (plain forward for 256 features, and for 96 in fp32, whose gated
               form needs it), the state handed on
  first_layer  the first layer's training step: swish and position encoding of queries and keys,
               attention with queries and keys twice as wide as values, and all gradients
  decode       one decode call: `S` tokens per sequence against the running states (with `lrpe`:
               the first layer's, whose queries and keys go through the input side first)

Sizes: the paper's models (8 / 16 / 32 heads of 128 features, 2048 and 8192 tokens), the long
sequences and the decode batch of the benchmark, the other head widths the library has, and the
odd lengths and small batches that serving meets.  Shapes are [Bt, H, N, D].
"""
import math

import torch

import paper_2307_14995_amd as ltn
from paper_2307_14995_amd import synth

EPS = 1e-6                       # under the root of the gate's norm
PREFIX = 1024                    # tokens behind a decode state or a carried prefill state
#: work of the largest listed case per pass, in token-heads x D^2 (bf16); fp32 products run at a
#: sixteenth of the bf16 matrix rate
BUDGET = 4 * 32 * 8192 * 128 ** 2
FP32_SHARE = 16


def _case(name, kind, Bt, H, N, D, dtype="bf16", decay="bench", state_in=False, lrpe=False):
    return {"name": name, "kind": kind, "Bt": Bt, "H": H, "N": N, "D": D, "dtype": dtype, "decay": decay,
            "state_in": state_in, "lrpe": lrpe}


def listed():
    return [
        # pre-training: the 7B-shaped layer at the paper's training length (the headline workload)
        _case("train_7b", "train", 4, 32, 8192, 128),
        # pre-training: the 385M-shaped layer
        _case("train_385m", "train", 8, 8, 2048, 128),
        # one long document, its length no multiple of anything
        _case("train_long", "train", 1, 32, 16301, 128),
        # wider heads at the 7B model's width
        _case("train_wide_heads", "train", 2, 16, 4096, 256),
        # heads of 96 features, packed documents of an odd length
        _case("train_heads96", "train", 8, 12, 1999, 96),
        # the full token mixer, 1B-shaped, Eq. 2's decays
        _case("mixer_1b", "mixer", 8, 16, 2048, 128, decay="paper"),
        # the full token mixer in fp32: numerics checks and small-model training
        _case("mixer_385m_fp32", "mixer", 4, 8, 2048, 128, dtype="fp32"),
        # the first layer of the 1B shape
        _case("first_layer_1b", "first_layer", 4, 16, 2048, 128),
        # serving: one user's prompt through a 7B-shaped layer
        _case("prefill_prompt", "prefill", 1, 32, 3001, 128),
        # serving: the next chunk of a few prompts, small heads
        _case("prefill_chunk", "prefill", 4, 8, 200, 64, state_in=True),
        # serving: one token for a full batch (the benchmark's decode workload)
        _case("decode_batch", "decode", 64, 32, 1, 128),
        # serving: one token for one user
        _case("decode_one", "decode", 1, 32, 1, 128),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(("train", "mixer", "prefill", "first_layer", "decode"), (30, 20, 20, 12, 18))[0]
    dtype = "fp32" if rng.random() < 0.25 else "bf16"
    lrpe = kind == "first_layer" or (kind == "decode" and rng.random() < 0.2)
    D = rng.choice((64, 128)) if lrpe else rng.choices((64, 96, 128, 256), (25, 15, 40, 20))[0]
    budget = BUDGET // (FP32_SHARE if dtype == "fp32" else 1)
    if kind == "mixer":
        budget = budget * 2 // 3     # three calls where training has two
    if kind == "first_layer":
        budget = budget // 3         # queries and keys twice as wide, and the input side
    H = rng.choice((4, 6, 8, 12, 16, 20, 24, 32, 40))
    if kind == "decode":
        most = BUDGET // (128 ** 2 * 512) // H * (128 * 128) // (D * D * (2 if lrpe else 1))
        Bt = _log_int(rng, 1, max(1, min(96, most)))
        N = rng.choice((1, 1, 1, 2, 3, 5, 8))
    else:
        while budget // (H * D * D) < 64:
            H //= 2
        # fp32 is for numerics checks and small models: sequences of the 2048-token context at most
        N = _log_int(rng, 16, min(2048 if dtype == "fp32" else 32768, budget // (H * D * D)))
        Bt = _log_int(rng, 1, max(1, min(32, budget // (H * D * D * N))))
    decay = rng.choice(("bench", "paper"))
    return {"kind": kind, "Bt": Bt, "H": H, "N": N, "D": D, "dtype": dtype, "decay": decay,
            "state_in": kind == "prefill" and rng.random() < 0.5, "lrpe": lrpe}


def _dtype(case):
    return torch.float32 if case["dtype"] == "fp32" else torch.bfloat16


def _gated(case):
    """Prefill runs the fused gated forward where the library has one without the stored output."""
    return case["D"] in (64, 128) or (case["D"] == 96 and case["dtype"] == "bf16")


def prepare(case, seed):
    Bt, H, N, D, kind = case["Bt"], case["H"], case["N"], case["D"], case["kind"]
    dt, dev = _dtype(case), torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)

    def randn(*shape, scale=1.0, dtype=dt):
        x = torch.randn(shape, generator=g, device=dev, dtype=dtype)
        return x.mul_(scale) if scale != 1.0 else x

    s = D ** -0.5
    lam = synth.decay_bench_rule(H) if case["decay"] == "bench" else synth.decay_paper_rule(H, 4, 16)
    st = {"case": case, "decay": lam.to(dev)}

    def state(rows):
        # the spread of a state behind PREFIX tokens of q, k, v ~ N(0,1)/sqrt(D)
        l2 = lam.double() ** 2
        var = (1 - l2 ** PREFIX) / (1 - l2) / (rows * D)
        return randn(Bt, H, rows, D, dtype=torch.float32).mul_(var.sqrt().float().to(dev).view(1, H, 1, 1))

    if kind == "decode":
        if case["lrpe"]:
            st.update(xq=randn(Bt, H, N, D), xk=randn(Bt, H, N, D), v=randn(Bt, H, N, D, scale=s),
                      theta=synth.make_theta(H, D, seed % 65536).to(dev), kv=state(2 * D))
        else:
            shape = (Bt, H, D) if N == 1 else (Bt, H, N, D)
            st.update(q=randn(*shape, scale=s), k=randn(*shape, scale=s), v=randn(*shape, scale=s), kv=state(D))
        return st
    st["v"] = randn(Bt, H, N, D, scale=s)
    if kind == "first_layer":
        st.update(xq=randn(Bt, H, N, D), xk=randn(Bt, H, N, D), d_o=randn(Bt, H, N, D),
                  theta=synth.make_theta(H, D, seed % 65536).to(dev))
        return st
    st.update(q=randn(Bt, H, N, D, scale=s), k=randn(Bt, H, N, D, scale=s))
    if kind == "train":
        st["d_o"] = randn(Bt, H, N, D)
    if kind == "mixer":
        st.update(u=randn(Bt, H, N, D), d_y=randn(Bt, H, N, D))
    if kind == "prefill":
        if _gated(case):
            st["u"] = randn(Bt, H, N, D)
        st["kv_in"] = state(D) if case["state_in"] else None
    return st


def run(st):
    case, decay = st["case"], st["decay"]
    kind = case["kind"]
    if kind == "train":
        o = ltn.ltn_attn_fwd(st["q"], st["k"], st["v"], decay)
        return (o, *ltn.ltn_attn_bwd(st["q"], st["k"], st["v"], st["d_o"], decay))
    if kind == "mixer":
        o, y = ltn.ltn_attn_fwd_gated(st["q"], st["k"], st["v"], st["u"], decay, eps=EPS)
        d_o, d_u = ltn.ltn_gate_bwd(o, st["u"], st["d_y"], eps=EPS)
        return (y, d_u, *ltn.ltn_attn_bwd(st["q"], st["k"], st["v"], d_o, decay))
    if kind == "prefill":
        if _gated(case):
            _, y, kv = ltn.ltn_attn_fwd_gated(st["q"], st["k"], st["v"], st["u"], decay, eps=EPS, kv_in=st["kv_in"],
                                              return_state=True, store_o=False)
        else:
            y, kv = ltn.ltn_attn_fwd(st["q"], st["k"], st["v"], decay, kv_in=st["kv_in"], return_state=True)
        return y, kv
    if kind == "first_layer":
        q = ltn.ltn_prologue_fwd(st["xq"], st["theta"])
        k = ltn.ltn_prologue_fwd(st["xk"], st["theta"])
        o = ltn.ltn_attn_fwd_dkdv(q, k, st["v"], decay)
        dq, dk, dv = ltn.ltn_attn_bwd_dkdv(q, k, st["v"], st["d_o"], decay)
        dxq, dth_q = ltn.ltn_prologue_bwd(st["xq"], dq, st["theta"])
        dxk, dth_k = ltn.ltn_prologue_bwd(st["xk"], dk, st["theta"])
        return o, dxq, dxk, dv, dth_q, dth_k
    if case["lrpe"]:
        q = ltn.ltn_prologue_fwd(st["xq"], st["theta"], pos0=PREFIX)
        k = ltn.ltn_prologue_fwd(st["xk"], st["theta"], pos0=PREFIX)
        return ltn.ltn_attn_decode_steps_dkdv(q, k, st["v"], st["kv"], decay), st["kv"]
    if st["q"].dim() == 3:
        return ltn.ltn_attn_decode_step(st["q"], st["k"], st["v"], st["kv"], decay), st["kv"]
    return ltn.ltn_attn_decode_steps(st["q"], st["k"], st["v"], st["kv"], decay), st["kv"]


def work(case):
    """Bytes: each entry point's inputs read once and its outputs written once, in units of one
    [Bt, H, N, D] tensor, plus the fp32 states.  Operations: the recurrent form's products (2 D^2
    per token to update a state, 2 D^2 to read it; the gradients five such products)."""
    Bt, H, N, D, kind = case["Bt"], case["H"], case["N"], case["D"], case["kind"]
    rows = Bt * H * N
    unit = rows * D * (4 if case["dtype"] == "fp32" else 2)
    state = Bt * H * D * D * 4
    if kind == "train":
        return {"bytes": (4 + 7) * unit, "flops": 14 * D * D * rows}
    if kind == "mixer":
        return {"bytes": (6 + 5 + 7) * unit, "flops": 14 * D * D * rows}
    if kind == "prefill":
        return {"bytes": (5 if _gated(case) else 4) * unit + (2 if case["state_in"] else 1) * state, "flops": 4 * D * D * rows}
    if kind == "first_layer":
        # 2 expansions (1 in, 2 out); forward 2+2+1 in, 1 out; backward 2+2+1+1 in, 2+2+1 out;
        # 2 derivatives of the expansion (1+2 in, 1 out)
        return {"bytes": (6 + 6 + 11 + 8) * unit, "flops": 28 * D * D * rows}
    if case["lrpe"]:
        return {"bytes": (6 + 6) * unit + 4 * state, "flops": 8 * D * D * rows}
    return {"bytes": 4 * unit + 2 * state, "flops": 4 * D * D * rows}


#: Largest errors against an fp64 evaluation of the same pass, over the listed cases but the largest
#: and 40 drawn ones, as (relative 2-norm, largest over max(rms, value)); the tolerance is four times that.
#:   fp32                     3.4e-7, 2.1e-5
#:   train, prefill bf16      2.7e-3, 3.5e-2
#:   mixer bf16               4.0e-3, 1.1e-1  (the gate's derivative divides by the norm of the stored, rounded O)
#:   first_layer bf16         4.0e-3, 5.7e-2; the angle gradients of short sequences 1.2e-2, 7.8e-2 (sums that cancel,
#:                            over terms rounded to bf16; 3e-2 is as much as is ever allowed)
#:   decode bf16              1.7e-3, 3.9e-3 (the output's own rounding); with lrpe 2.3e-3, 2.5e-2
TOLERANCE = {
    "fp32": {"rel": 1.4e-6, "max": 1e-4},
    "train": {"rel": 1.1e-2, "max": 0.14},
    "prefill": {"rel": 1.1e-2, "max": 0.14},
    "mixer": {"rel": 1.6e-2, "max": 0.42},
    "first_layer": {"rel": 3e-2, "max": 0.3},
    "decode": {"rel": 7e-3, "max": 0.016},
    "decode_lrpe": {"rel": 9e-3, "max": 0.1},
}


def tolerance(case):
    if case["dtype"] == "fp32":
        return dict(TOLERANCE["fp32"])
    return dict(TOLERANCE["decode_lrpe" if case["kind"] == "decode" and case["lrpe"] else case["kind"]])
