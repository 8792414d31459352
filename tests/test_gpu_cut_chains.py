"""bf16 passes in a few more workgroups than the GPU has compute units: the chains whose last pass
runs in two parts (the second starting from the first's state, kept in the output's own rows).

The parts add the same terms in the same order as the whole chain, so every result must be the same bits as
with the cut switched off; the chains on both sides of the line between cut and whole ones are held to
the fp64 oracle as well."""
import pytest
import torch

import paper_2307_14995_amd as ltn
from paper_2307_14995_amd import synth
from oracle import ltn_oracle as orc
from _helpers import TOL, check, force_segs, gpu, mixed_decay

pytestmark = pytest.mark.gpu

BF = torch.bfloat16
# (D, Bt, H, N, cut chains, of the gated forward too): 257 .. 384 workgroups in two rounds and 520 .. 640 in three,
# chain counts that are multiples of 8 and not (their ids are dealt differently), the shortest length that is cut
# (second parts of 321 tokens, 577 of 256 features) and a ragged one, last rounds exactly half full (384 and 640); plain
# forwards of small inputs run whole
FORWARD = [(64, 4, 65, 705, 0, 4), (64, 3, 96, 1090, 0, 32), (64, 5, 105, 769, 13, 13), (96, 1, 257, 705, 0, 1),
           (96, 8, 40, 1100, 64, 64), (128, 3, 99, 705, 41, 41), (128, 4, 66, 900, 8, 8), (128, 1, 530, 770, 18, 18),
           (256, 5, 13, 1217, 1, 0), (256, 5, 16, 1300, 16, 0), (256, 3, 50, 1217, 22, 0),
           (64, 4, 65, 1300, 4, 4), (64, 3, 96, 1500, 32, 32), (96, 1, 257, 900, 1, 1), (96, 4, 96, 800, 128, 128),
           (128, 1, 383, 705, 127, 127), (64, 8, 80, 705, 128, 128)]
# (D, Bt, H, N, cut chains); the first of 64 features and 128, 8, 15, 900 are too small; last rounds exactly half full
# on either side of the line, and of chains of 512 KiB
BACKWARD = [(64, 1, 86, 705, 0), (64, 8, 14, 1000, 0), (96, 8, 12, 1090, 32), (96, 3, 31, 705, 23), (128, 5, 20, 705, 44),
            (128, 8, 15, 900, 0), (256, 1, 22, 1217, 2), (256, 2, 16, 1250, 32),
            (64, 1, 86, 1100, 2), (64, 8, 14, 1500, 80), (128, 8, 15, 1100, 104), (128, 4, 32, 1450, 128),
            (128, 4, 32, 1300, 0), (128, 4, 32, 2048, 0), (128, 4, 32, 2080, 128), (128, 1, 128, 2625, 128)]


def lines(chains, cut):
    return sorted({0, max(cut - 1, 0), min(cut, chains - 1), chains - 1})


def is_cut(Bt, H, N, D, call, chains, Dv=None):
    """The library's own word for it: so many chains in two parts (with whole chains forced none)."""
    with force_segs(1):
        assert ltn.ltn_attn_query_cut(Bt, H, N, D, Dv or D, BF, call)[0] == 0
    return ltn.ltn_attn_query_cut(Bt, H, N, D, Dv or D, BF, call)[0] == chains


def some(t, chains, keep):
    return t.reshape(1, chains, *t.shape[2:])[:, keep]


@pytest.mark.parametrize("D,Bt,H,N,cut", [c[:5] for c in FORWARD])
def test_forward(D, Bt, H, N, cut):
    assert is_cut(Bt, H, N, D, 0, cut)
    q, k, v = synth.make_qkv(Bt, H, N, D, BF, 900 + N)
    decay = mixed_decay(H)
    kv0 = torch.randn(Bt, H, D, D, generator=torch.Generator().manual_seed(N)) / D
    args = gpu(q, k, v, decay)
    with force_segs(1):
        o_whole, kv_whole = ltn.ltn_attn_fwd(*args, kv_in=kv0.cuda(), return_state=True)
    state = kv0.cuda()
    o, kv = ltn.ltn_attn_fwd(*args, kv_in=state, kv_out=state)
    assert torch.equal(o, o_whole) and torch.equal(kv, kv_whole)
    assert torch.equal(ltn.ltn_attn_fwd(*args, kv_in=kv0.cuda()), o_whole)
    keep = lines(Bt * H, cut)
    o_ref, kv_ref = orc.fwd_recurrent(*(some(t, Bt * H, keep) for t in (q, k, v)), decay.repeat(Bt)[keep],
                                      kv_in=some(kv0, Bt * H, keep), return_state=True)
    check("O", some(o, Bt * H, keep), o_ref, TOL[BF])
    check("kv", some(kv, Bt * H, keep), kv_ref, TOL[BF])


@pytest.mark.parametrize("D,Bt,H,N,cut", [(*c[:4], c[5]) for c in FORWARD if c[0] != 256])
def test_gated_forward(D, Bt, H, N, cut):
    """The state passes through y's rows, whether o is stored or not."""
    assert is_cut(Bt, H, N, D, 2, cut)
    q, k, v = synth.make_qkv(Bt, H, N, D, BF, 920 + N)
    u = synth.make_gate(Bt, H, N, D, BF, 920 + N)
    decay = mixed_decay(H)
    kv0 = torch.randn(Bt, H, D, D, generator=torch.Generator().manual_seed(N)) / D
    args = gpu(q, k, v, u, decay)

    def call(store_o):
        return ltn.ltn_attn_fwd_gated(*args, eps=1e-6, kv_in=kv0.cuda(), return_state=True, store_o=store_o)

    with force_segs(1):
        o_whole, y_whole, kv_whole = call(True)
        _, y_alone, _ = call(False)
    o, y, kv = call(True)
    assert torch.equal(o, o_whole) and torch.equal(y, y_whole) and torch.equal(kv, kv_whole)
    _, y, kv = call(False)
    assert torch.equal(y, y_alone) and torch.equal(kv, kv_whole)
    keep = lines(Bt * H, cut)
    o_ref, kv_ref = orc.fwd_recurrent(*(some(t, Bt * H, keep) for t in (q, k, v)), decay.repeat(Bt)[keep],
                                      kv_in=some(kv0, Bt * H, keep), return_state=True)
    check("O", some(o, Bt * H, keep), o_ref, TOL[BF])
    check("Y", some(y, Bt * H, keep), orc.gate_fwd(o_ref, some(u, Bt * H, keep), 1e-6), TOL[BF])
    check("kv", some(kv, Bt * H, keep), kv_ref, TOL[BF])


@pytest.mark.parametrize("D,Bt,H,N,cut", BACKWARD)
def test_backward(D, Bt, H, N, cut):
    assert is_cut(Bt, H, N, D, 1, cut)
    q, k, v = synth.make_qkv(Bt, H, N, D, BF, 950 + N)
    g = synth.make_do(Bt, H, N, D, BF, 950 + N)
    decay = mixed_decay(H)
    args = gpu(q, k, v, g, decay)
    with force_segs(1):
        whole = ltn.ltn_attn_bwd(*args)
    grads = ltn.ltn_attn_bwd(*args)
    assert all(torch.equal(x, y) for x, y in zip(grads, whole))
    keep = lines(Bt * H, cut)
    refs = orc.bwd_recurrent(*(some(t, Bt * H, keep) for t in (q, k, v, g)), decay.repeat(Bt)[keep])
    for n, x, r in zip(("dQ", "dK", "dV"), grads, refs):
        check(n, some(x, Bt * H, keep), r, TOL[BF])


# (Dk, Dv, Bt, H, N, chains cut in the forward and dV (the second part of dV's reversed token axis lies in front),
# of dQ's)
@pytest.mark.parametrize("Dk,Dv,Bt,H,N,cut,cut_q", [(256, 128, 2, 65, 1217, 2, 4), (256, 128, 9, 16, 1300, 16, 32),
                                                    (256, 128, 4, 18, 705, 0, 16), (128, 64, 4, 65, 705, 0, 0),
                                                    (128, 64, 3, 96, 800, 32, 0), (128, 64, 8, 10, 705, 0, 32),
                                                    (128, 64, 3, 30, 770, 0, 52), (128, 64, 4, 65, 780, 4, 0)])
def test_unequal_widths(Dk, Dv, Bt, H, N, cut, cut_q):
    assert is_cut(Bt, H, N, Dk, 0, cut, Dv) and is_cut(Bt, H, N, Dk, 1, cut_q, Dv)
    q, k, v = synth.make_qkv_dkdv(Bt, H, N, Dk, Dv, BF, 70 + N)
    g = synth.make_do(Bt, H, N, Dv, BF, 70 + N)
    decay = mixed_decay(H)
    kv0 = torch.randn(Bt, H, Dk, Dv, generator=torch.Generator().manual_seed(N)) / Dk
    args, do = gpu(q, k, v), g.cuda()
    with force_segs(1):
        whole = [*ltn.ltn_attn_fwd_dkdv(*args, decay.cuda(), kv_in=kv0.cuda(), return_state=True),
                 *ltn.ltn_attn_bwd_dkdv(*args, do, decay.cuda())]
    got = [*ltn.ltn_attn_fwd_dkdv(*args, decay.cuda(), kv_in=kv0.cuda(), return_state=True),
           *ltn.ltn_attn_bwd_dkdv(*args, do, decay.cuda())]
    assert all(torch.equal(x, y) for x, y in zip(got, whole))
    keep = [0, Bt * H - 1]
    ins = [some(t, Bt * H, keep) for t in (q, k, v)]
    refs = [*orc.fwd_recurrent_dkdv(*ins, decay.repeat(Bt)[keep], kv_in=some(kv0, Bt * H, keep), return_state=True),
            *orc.bwd_recurrent_dkdv(*ins, some(g, Bt * H, keep), decay.repeat(Bt)[keep])]
    for n, x, r in zip(("O", "kv", "dQ", "dK", "dV"), got, refs):
        check(n, some(x, Bt * H, keep), r, TOL[BF])


def test_outputs_inside_larger_buffers():
    """The states and flags that pass through the output's rows stay inside them."""
    D, Bt, H, N = 96, 8, 12, 1090
    assert is_cut(Bt, H, N, D, 1, 32)
    q, k, v = synth.make_qkv(Bt, H, N, D, BF, 31)
    g = synth.make_do(Bt, H, N, D, BF, 31)
    decay = synth.decay_bench_rule(H)
    guard = 4096
    raws = [torch.full((q.numel() + 2 * guard,), 7.0, device="cuda", dtype=BF) for _ in range(3)]
    outs = [r[guard:guard + q.numel()].view_as(q) for r in raws]
    args = gpu(q, k, v, g, decay)
    ltn.ltn_attn_bwd(*args, out=outs)
    with force_segs(1):
        whole = ltn.ltn_attn_bwd(*args)
    for x, y, raw in zip(outs, whole, raws):
        assert torch.equal(x, y)
        assert bool((raw[:guard] == 7.0).all()) and bool((raw[-guard:] == 7.0).all())


def test_replayed_graph():
    """Captured once and replayed over changing inputs, with eager calls in between: every replay waits for its own
    states (the flags are cleared by a kernel of the call)."""
    D, Bt, H, N = 128, 5, 20, 770          # 44 of the 100 chains
    assert is_cut(Bt, H, N, D, 1, 44)
    decay = synth.decay_bench_rule(H).cuda()
    q, k, v, g = (torch.empty(Bt, H, N, D, device="cuda", dtype=BF) for _ in range(4))

    def fill(seed):
        for x, y in zip((q, k, v, g), (*synth.make_qkv(Bt, H, N, D, BF, seed), synth.make_do(Bt, H, N, D, BF, seed))):
            x.copy_(y)

    def call():
        return ltn.ltn_attn_bwd(q, k, v, g, decay)

    fill(1)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = call()
    for seed in (2, 3, 4):
        fill(seed)
        graph.replay()
        torch.cuda.synchronize()
        got = [x.clone() for x in captured]
        with force_segs(1):
            whole = call()
        assert all(torch.equal(x, y) for x, y in zip(got, whole))


def same(x, y):
    return torch.equal(x.isnan(), y.isnan()) and torch.equal(x.nan_to_num(), y.nan_to_num())


@pytest.mark.parametrize("token", [100, 447, 448, 600])
def test_infinite_token_on_either_side_of_the_cut(token):
    """Cut at 448 (dQ walks from the first token): Inf and NaN appear where they do in whole chains, in the
    outputs, in the state that passes through them and in the returned state."""
    D, Bt, H, N = 128, 5, 20, 770
    assert is_cut(Bt, H, N, D, 1, 44) and ltn.ltn_attn_query_cut(Bt, H, N, D, D, BF, 1)[1] == 448
    q, k, v = synth.make_qkv(Bt, H, N, D, BF, 41)
    g = synth.make_do(Bt, H, N, D, BF, 41)
    k[..., token, 5] = float("inf")
    args = gpu(q, k, v, g, mixed_decay(H))
    with force_segs(1):
        whole = ltn.ltn_attn_bwd(*args)
    grads = ltn.ltn_attn_bwd(*args)
    assert all(same(x, y) for x, y in zip(grads, whole))
    # (within the token's own block of 64, masked scores are zeros: 0 x Inf there, as in whole chains)
    finite = grads[0].isfinite().all(-1)
    assert bool(finite[..., :token // 64 * 64].all()) and not bool(finite[..., token:].all())


@pytest.mark.parametrize("token", [100, 600])
def test_infinite_token_and_state_in_a_gated_forward(token):
    D, Bt, H, N = 128, 3, 99, 705
    assert is_cut(Bt, H, N, D, 2, 41) and is_cut(Bt, H, N, D, 0, 41)
    q, k, v = synth.make_qkv(Bt, H, N, D, BF, 43)
    k[:, ::2, token, 5] = float("inf")
    kv0 = torch.zeros(Bt, H, D, D)
    kv0[:, 1::2, 3, 7] = float("-inf")
    args, u = gpu(q, k, v), synth.make_gate(Bt, H, N, D, BF, 43).cuda()
    decay = mixed_decay(H).cuda()

    def calls():
        return [*ltn.ltn_attn_fwd(*args, decay, kv_in=kv0.cuda(), return_state=True),
                *ltn.ltn_attn_fwd_gated(*args, u, decay, eps=1e-6, kv_in=kv0.cuda(), return_state=True)]

    with force_segs(1):
        whole = calls()
    got = calls()
    assert all(same(x, y) for x, y in zip(got, whole))
    finite = bool(got[1].isfinite().all())
    assert not finite


def test_two_streams():
    """Cut launches of two streams in flight at once: each waits for its own states."""
    D, Bt, H, N = 96, 8, 12, 1090
    assert is_cut(Bt, H, N, D, 1, 32)
    decay = synth.decay_bench_rule(H).cuda()
    ins = [gpu(*synth.make_qkv(Bt, H, N, D, BF, s), synth.make_do(Bt, H, N, D, BF, s)) for s in (51, 52)]
    with force_segs(1):
        whole = [ltn.ltn_attn_bwd(*x, decay) for x in ins]
    streams = [torch.cuda.Stream() for _ in ins]
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    got = [[], []]
    for _ in range(4):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                got[i].append(ltn.ltn_attn_bwd(*ins[i], decay))
    torch.cuda.synchronize()
    for w, each in zip(whole, got):
        for grads in each:
            assert all(torch.equal(x, y) for x, y in zip(grads, w))
