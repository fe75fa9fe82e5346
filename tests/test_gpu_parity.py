"""HIP path vs the fp64 oracle on the same seeded inputs (needs an MI355X).

Bar: max relative Frobenius error per (sequence, value head) <= 2e-3 for
states and <= 5e-3 for output blocks.  Small cases span several chunks and a
ragged tail; the workload cases run at full size in the launch configuration
the benchmark times, checked in full where the oracle finishes in seconds and
on sampled (layer, head) units otherwise.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_30310_amd as gdn
import synth
from synth import workloads
from tests.gpu_util import (OUTPUT_TOL, STATE_TOL, device_inputs, first_half_share, oracle_run, output_err, slow_decay,
                            state_err, to_f64)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    gdn.load_library()


def _report(name, **errs):
    print(f"[parity] {name}: " + ", ".join(f"{k}={v:.3e}" for k, v in errs.items()), flush=True)


LENS = [0, 1, 63, 64, 65, 127, 128, 205]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 128), (64, 128), (128, 64)])
@pytest.mark.parametrize("grp", [1, 2])
def test_ragged_varlen(dtype, dk, dv, grp):
    shape = synth.Shape(hk=2, hv=2 * grp, dk=dk, dv=dv, dtype=dtype)
    seqs = [synth.tokens(100, 0, i, 0, n, shape) for i, n in enumerate(LENS)]
    p = synth.pack(seqs)
    x = device_inputs(p)
    st = gdn.tail_replay(x["k"], x["v"], x["g"], x["beta"], x["cu"], x["cu_host"])
    _, want = oracle_run(p)
    e_tail = state_err(to_f64(st), want)
    rng = np.random.default_rng(7)
    s0 = (rng.standard_normal((len(LENS), shape.hv, dk, dv)) * 0.3).astype(np.float32)
    o, st2 = gdn.chunk_forward(x["q"], x["k"], x["v"], x["g"], x["beta"], x["cu"], x["cu_host"],
                               state_in=torch.from_numpy(s0).cuda(), scale=0.5)
    wo, ws = oracle_run(p, state_in=s0.astype(np.float64), outputs=True, scale=0.5)
    e_st = state_err(to_f64(st2), ws)
    e_o = output_err(to_f64(o), wo, p.cu_seqlens)
    _report(f"ragged {dtype} dk={dk} dv={dv} grp={grp}", tail=e_tail, fwd_state=e_st, out=e_o)
    assert e_tail <= STATE_TOL and e_st <= STATE_TOL and e_o <= OUTPUT_TOL
    # the empty sequence: zero state after replay, state_in after forward
    assert torch.count_nonzero(st[0]).item() == 0
    assert torch.equal(st2[0], torch.from_numpy(s0[0]).cuda())


# Batches of 4 value heads beyond the chip.  72 short sequences: tails run in
# rounds of 64 columns, fp32 ones of d_v = 128 a head per workgroup; forwards a
# head per workgroup with a peeled last round (bf16, d_v = 128), in 64 columns
# (bf16, d_v = 64) or in 32 (fp32).  220 sequences of three chunks: bf16 tails
# run the wide scan (two 16-column tiles per wave) at every (d_k, d_v), with a
# peeled last round.
WIDE_LENS = [1 + (37 * i) % 200 for i in range(72)]
EVEN_LENS = [129 + (37 * i) % 64 for i in range(220)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 128), (64, 128), (128, 64)])
@pytest.mark.parametrize("lens", [WIDE_LENS, EVEN_LENS], ids=["ragged", "even"])
def test_batches_beyond_the_chip(dtype, dk, dv, lens):
    shape = synth.Shape(hk=2, hv=4, dk=dk, dv=dv, dtype=dtype)
    seqs = [synth.tokens(101, 0, i, 0, n, shape) for i, n in enumerate(lens)]
    p = synth.pack(seqs)
    x = device_inputs(p)
    st = gdn.tail_replay(x["k"], x["v"], x["g"], x["beta"], x["cu"], x["cu_host"])
    _, want = oracle_run(p)
    e_tail = state_err(to_f64(st), want)
    rng = np.random.default_rng(8)
    s0 = (rng.standard_normal((len(lens), shape.hv, dk, dv)) * 0.3).astype(np.float32)
    o, st2 = gdn.chunk_forward(x["q"], x["k"], x["v"], x["g"], x["beta"], x["cu"], x["cu_host"],
                               state_in=torch.from_numpy(s0).cuda(), scale=0.5)
    wo, ws = oracle_run(p, state_in=s0.astype(np.float64), outputs=True, scale=0.5)
    e_st = state_err(to_f64(st2), ws)
    e_o = output_err(to_f64(o), wo, p.cu_seqlens)
    _report(f"{len(lens)} sequences {dtype} dk={dk} dv={dv}", tail=e_tail, fwd_state=e_st, out=e_o)
    assert e_tail <= STATE_TOL and e_st <= STATE_TOL and e_o <= OUTPUT_TOL


# Tail replay in two halves: bf16 inputs with at least 20 chunks in the longest sequence
# and N x Hv x 8 <= 256 workgroups (d = 128).  Lengths cover an empty
# sequence, one token, two chunks (the second half one chunk), 7 chunks and 21
# with a ragged end, so every part meets a short or empty range somewhere.
# With the synthetic gates' usual decay the first half's share of the final
# state is ~1e-7 or less at these lengths and a wrong combine would pass
# unseen, so these inputs decay slowly (gate scale 0.002, beta x 0.1): the
# oracle itself shows the first half's share above 10%.
SPLIT_LENS = [0, 1, 70, 400, 1300]


@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 128), (64, 128), (128, 64)])
def test_split_tail_replay_ragged(dk, dv):
    shape = synth.Shape(hk=2, hv=4, dk=dk, dv=dv, dtype="bf16")
    seqs = [slow_decay(synth.tokens(102, 0, i, 0, n, shape, gate_scale=0.002))
            for i, n in enumerate(SPLIT_LENS)]
    p = synth.pack(seqs)
    x = device_inputs(p)
    st = gdn.tail_replay(x["k"], x["v"], x["g"], x["beta"], x["cu"], x["cu_host"])
    _, want = oracle_run(p)
    share = first_half_share(seqs[-1])
    e = state_err(to_f64(st), want)
    _report(f"split bf16 dk={dk} dv={dv}", tail=e, first_half_share=share)
    assert share > 0.1
    assert e <= STATE_TOL
    assert torch.count_nonzero(st[0]).item() == 0


def _chain(shape, hits, outputs_scale=1.0):
    """GPU: tail replay then suffix forward from the rebuilt state; the oracle
    does the same chain in fp64.  Returns the error triple."""
    tails = synth.pack([h.tail(shape) for h in hits])
    sufs = synth.pack([h.suffix(shape) for h in hits])
    xt = device_inputs(tails)
    xs = device_inputs(sufs)
    st = gdn.tail_replay(xt["k"], xt["v"], xt["g"], xt["beta"], xt["cu"], xt["cu_host"])
    o, st2 = gdn.chunk_forward(xs["q"], xs["k"], xs["v"], xs["g"], xs["beta"], xs["cu"],
                               xs["cu_host"], state_in=st, scale=outputs_scale)
    _, w_tail = oracle_run(tails)
    w_o, w_st = oracle_run(sufs, state_in=w_tail, outputs=True, scale=outputs_scale)
    return (state_err(to_f64(st), w_tail), state_err(to_f64(st2), w_st),
            output_err(to_f64(o), w_o, sufs.cu_seqlens))


def test_workload1_fused_replay_forward():
    # the bench configuration through the fused entry point, against the oracle
    shape, hits = workloads.workload1(819)
    tails = synth.pack([h.tail(shape) for h in hits])
    sufs = synth.pack([h.suffix(shape) for h in hits])
    xt, xs = device_inputs(tails), device_inputs(sufs)
    o, mid, st = gdn.replay_forward(xt["k"], xt["v"], xt["g"], xt["beta"], xt["cu"],
                                    xs["q"], xs["k"], xs["v"], xs["g"], xs["beta"], xs["cu"],
                                    cu_tail_host=xt["cu_host"], cu_suf_host=xs["cu_host"])
    _, w_tail = oracle_run(tails)
    w_o, w_st = oracle_run(sufs, state_in=w_tail, outputs=True)
    e = (state_err(to_f64(mid), w_tail), state_err(to_f64(st), w_st),
         output_err(to_f64(o), w_o, sufs.cu_seqlens))
    _report("workload1 fused r=819", tail=e[0], fwd_state=e[1], out=e[2])
    assert e[0] <= STATE_TOL and e[1] <= STATE_TOL and e[2] <= OUTPUT_TOL


def test_workload0_small_fp32():
    shape, hits = workloads.workload0()
    e = _chain(shape, hits)
    _report("workload0 r=205 s=256", tail=e[0], final=e[1], out=e[2])
    assert e[0] <= STATE_TOL and e[1] <= STATE_TOL and e[2] <= OUTPUT_TOL


@pytest.mark.parametrize("r", [410, 819])
def test_workload1_hybrid_shapes(r):
    shape, hits = workloads.workload1(r)
    e = _chain(shape, hits)
    _report(f"workload1 r={r} s=512", tail=e[0], final=e[1], out=e[2])
    assert e[0] <= STATE_TOL and e[1] <= STATE_TOL and e[2] <= OUTPUT_TOL


def test_workload3_varlen_hits():
    draw = workloads.workload3_draw()
    rs = [gdn.replay_len(m, ratio) for m, ratio, _ in draw]
    assert rs == [oracle.replay_len(m, ratio) for m, ratio, _ in draw]
    shape, hits = workloads.workload3(rs)
    e = _chain(shape, hits)
    _report("workload3 16 hits", tail=e[0], final=e[1], out=e[2])
    assert e[0] <= STATE_TOL and e[1] <= STATE_TOL and e[2] <= OUTPUT_TOL


def _head_slice(p, h, grp):
    """One value head's inputs (and its key head) as a Hk = Hv = 1 problem."""
    ex = p.exact()
    kh = h // grp
    return (ex["k"][:, kh:kh + 1], ex["v"][:, h:h + 1], ex["g"][:, h:h + 1],
            ex["beta"][:, h:h + 1], ex["cu_seqlens"], ex["q"][:, kh:kh + 1])


def test_workload2_layer_stack_sampled():
    """The 36-layer stack (prefix 32768, tail 3277, suffix 1024) in both launch
    forms the benchmark times: per layer, the tail replay (split in two
    halves at this length) then the suffix forward from the rebuilt state; and
    the 36 layers as one batched tail replay (the wide column scan, 36 x 52
    chunks in one launch) then one batched suffix forward (the whole-head
    scan).  Sampled (layer, value head) units against the oracle: the rebuilt
    state, the suffix outputs and the final state."""
    shape, hits = workloads.workload2()
    grp = shape.hv // shape.hk
    sample_layers = [0, 17, 35]
    sample_heads = [0, 13, 31]
    drawn = workloads.draw_hits(hits, shape)
    tails = synth.pack([t for t, _ in drawn])
    sufs = synth.pack([s for _, s in drawn])
    xt, xs = device_inputs(tails), device_inputs(sufs)
    r, s = hits[0].r, hits[0].s
    L = len(hits)
    # per layer, as benchmarked
    cu_t = torch.tensor([0, r], dtype=torch.int32)
    cu_s = torch.tensor([0, s], dtype=torch.int32)
    mid = torch.empty((L, shape.hv, 128, 128), dtype=torch.float32, device="cuda:0")
    fin = torch.empty_like(mid)
    o = torch.empty((L * s, shape.hv, 128), dtype=torch.bfloat16, device="cuda:0")
    for l in range(L):
        a, b = l * r, (l + 1) * r
        gdn.tail_replay(xt["k"][a:b], xt["v"][a:b], xt["g"][a:b], xt["beta"][a:b], cu_t.cuda(), cu_t,
                        state_out=mid[l:l + 1])
        a, b = l * s, (l + 1) * s
        gdn.chunk_forward(xs["q"][a:b], xs["k"][a:b], xs["v"][a:b], xs["g"][a:b], xs["beta"][a:b], cu_s.cuda(),
                          cu_s, state_in=mid[l:l + 1], o=o[a:b], state_out=fin[l:l + 1])
    # batched
    midb = gdn.tail_replay(xt["k"], xt["v"], xt["g"], xt["beta"], xt["cu"], xt["cu_host"])
    ob, finb = gdn.chunk_forward(xs["q"], xs["k"], xs["v"], xs["g"], xs["beta"], xs["cu"], xs["cu_host"],
                                 state_in=midb)
    torch.cuda.synchronize()
    got = {name: to_f64(t) for name, t in (("mid", mid), ("fin", fin), ("o", o), ("midb", midb),
                                            ("finb", finb), ("ob", ob))}
    worst = dict(mid=0.0, fin=0.0, out=0.0, midb=0.0, finb=0.0, outb=0.0)
    for l in sample_layers:
        tp, sp = synth.pack([drawn[l][0]]), synth.pack([drawn[l][1]])
        for h in sample_heads:
            k, v, g, b, cu, _ = _head_slice(tp, h, grp)
            _, w_mid = oracle.recurrence(k, v, g, b, cu)
            k2, v2, g2, b2, cu2, q2 = _head_slice(sp, h, grp)
            w_o, w_fin = oracle.recurrence(k2, v2, g2, b2, cu2, q=q2, state_in=w_mid)
            rows = slice(l * s, (l + 1) * s)
            for tag in ("", "b"):
                worst["mid" + tag] = max(worst["mid" + tag], state_err(got["mid" + tag][l:l + 1, h:h + 1], w_mid))
                worst["fin" + tag] = max(worst["fin" + tag], state_err(got["fin" + tag][l:l + 1, h:h + 1], w_fin))
                worst["out" + tag] = max(worst["out" + tag],
                                         output_err(got["o" + tag][rows, h:h + 1], w_o, cu2))
    _report("workload2 36 layers r=3277 s=1024 (sampled)", **worst)
    assert max(worst["mid"], worst["fin"], worst["midb"], worst["finb"]) <= STATE_TOL
    assert max(worst["out"], worst["outb"]) <= OUTPUT_TOL


def _bound_check(st_full, st_tail, st_head, g_tail, slack):
    """Per value head: ||S_full - S_tail||_F <= ||S_head||_F prod(alpha) + slack
    ||S_full||_F, prod(alpha) = exp(sum of g over the tail) (the attenuation
    bound of the replay).  Returns (max relative distance, max relative bound,
    heads where it fails)."""
    hv = st_full.shape[1]
    full = st_full[0].reshape(hv, -1)
    dist = np.linalg.norm(full - st_tail[0].reshape(hv, -1), axis=1)
    nf = np.linalg.norm(full, axis=1)
    bound = np.linalg.norm(st_head[0].reshape(hv, -1), axis=1) * np.exp(g_tail.sum(axis=0))
    bad = [h for h in range(hv) if dist[h] > bound[h] + slack * nf[h]]
    return float((dist / nf).max()), float((bound / nf).max()), bad


@pytest.mark.parametrize("gate_scale", workloads.WORKLOAD4_GATE_SCALES)
def test_workload4_full_prefill_and_tails_sampled(gate_scale):
    shape, hit = workloads.workload4(3277, gate_scale)
    grp = shape.hv // shape.hk
    full = synth.pack([hit.prefix(shape)])
    x = device_inputs(full)
    o, st_full = gdn.chunk_forward(x["q"], x["k"], x["v"], x["g"], x["beta"], x["cu"],
                                   x["cu_host"])
    got_st = to_f64(st_full)
    heads = [5, 26]
    e_st = e_o = 0.0
    for h in heads:
        k, v, g, b, cu, q = _head_slice(full, h, grp)
        w_o, w_st = oracle.recurrence(k, v, g, b, cu, q=q)
        e_st = max(e_st, state_err(got_st[:, h:h + 1], w_st))
        got_o = to_f64(o[:, h:h + 1])
        e_o = max(e_o, output_err(got_o, w_o, cu))
    e_tail = 0.0
    m = hit.m
    bound_rows = []
    for r in workloads.WORKLOAD4_TAILS:
        _, hr = workloads.workload4(r, gate_scale)
        tp = synth.pack([hr.tail(shape)])
        xt = device_inputs(tp)
        st = to_f64(gdn.tail_replay(xt["k"], xt["v"], xt["g"], xt["beta"], xt["cu"],
                                    xt["cu_host"]))
        for h in heads:
            k, v, g, b, cu, _ = _head_slice(tp, h, grp)
            _, want = oracle.recurrence(k, v, g, b, cu)
            e_tail = max(e_tail, state_err(st[:, h:h + 1], want))
        # the replay's attenuation bound on the GPU results, every value head:
        # S_head is the full-prefill state at m - r (the head of the prefix,
        # replayed from zero); slack for the two states' parity errors
        cu_h = torch.tensor([0, m - r], dtype=torch.int32)
        st_head = to_f64(gdn.tail_replay(x["k"][:m - r], x["v"][:m - r], x["g"][:m - r], x["beta"][:m - r],
                                         cu_h.cuda(), cu_h))
        rel, rel_bound, bad = _bound_check(got_st, st, st_head, full.g[m - r:].astype(np.float64), 2 * STATE_TOL)
        bound_rows.append((r, rel, rel_bound))
        assert not bad, f"bound fails at r={r} for heads {bad}"
    print(f"[bound] gate scale {gate_scale}: " + "; ".join(
        f"r={r}: |S_full-S_tail|/|S_full| max {rel:.2e} <= bound max {rb:.2e}" for r, rel, rb in bound_rows),
        flush=True)
    _report(f"workload4 s={gate_scale} full 32K + tails (sampled)", full_state=e_st,
            full_out=e_o, tails=e_tail)
    assert e_st <= STATE_TOL and e_o <= OUTPUT_TOL and e_tail <= STATE_TOL


@pytest.mark.parametrize("seed", range(12))
def test_random_configurations(seed):
    """Fixed-seed random configurations of every call with a state or output:
    1-12 sequences of 0-400 tokens (empty and one-token sequences included by
    chance and by force), d_k, d_v in {64, 128}, 1-4 value heads per key head,
    bf16 or fp32, tail replay, forward from a random state and the fused call."""
    rng = np.random.default_rng(1000 + seed)
    dk, dv = int(rng.choice([64, 128])), int(rng.choice([64, 128]))
    hk = int(rng.integers(1, 4))
    grp = int(rng.choice([1, 2, 4]))
    dtype = "bf16" if rng.random() < 0.7 else "f32"
    shape = synth.Shape(hk=hk, hv=hk * grp, dk=dk, dv=dv, dtype=dtype)
    n = int(rng.integers(1, 13))
    lens = [int(x) for x in rng.integers(0, 401, n)]
    lens[int(rng.integers(0, n))] = int(rng.choice([0, 1, 64]))
    gate = float(rng.choice([0.02, 0.1, 0.5]))
    tail = synth.pack([synth.tokens(300 + seed, 0, i, 0, L, shape, gate) for i, L in enumerate(lens)], shape)
    suf_lens = [int(x) for x in rng.integers(0, 200, n)]
    suf = synth.pack([synth.tokens(300 + seed, 0, i, L, L + s, shape, gate)
                      for i, (L, s) in enumerate(zip(lens, suf_lens))], shape)
    xt, xs = device_inputs(tail), device_inputs(suf)
    scale = dk ** -0.5
    st = gdn.tail_replay(xt["k"], xt["v"], xt["g"], xt["beta"], xt["cu"], xt["cu_host"])
    _, want_st = oracle_run(tail)
    e_tail = state_err(to_f64(st), want_st)
    s0 = (rng.standard_normal((n, shape.hv, dk, dv)) * 0.2).astype(np.float32)
    o, st2 = gdn.chunk_forward(xs["q"], xs["k"], xs["v"], xs["g"], xs["beta"], xs["cu"], xs["cu_host"],
                               state_in=torch.from_numpy(s0).cuda(), scale=scale)
    want_o, want_st2 = oracle_run(suf, state_in=s0.astype(np.float64), outputs=True, scale=scale)
    e_fwd, e_out = state_err(to_f64(st2), want_st2), output_err(to_f64(o), want_o, suf.cu_seqlens)
    o3, mid, fin = gdn.replay_forward(xt["k"], xt["v"], xt["g"], xt["beta"], xt["cu"], xs["q"], xs["k"],
                                      xs["v"], xs["g"], xs["beta"], xs["cu"], cu_tail_host=xt["cu_host"],
                                      cu_suf_host=xs["cu_host"], scale=scale)
    want_o3, want_fin = oracle_run(suf, state_in=want_st, outputs=True, scale=scale)
    e_mid, e_fin = state_err(to_f64(mid), want_st), state_err(to_f64(fin), want_fin)
    e_out3 = output_err(to_f64(o3), want_o3, suf.cu_seqlens)
    _report(f"random {seed}: N={n} {dtype} dk={dk} dv={dv} hk={hk} grp={grp} gate={gate}",
            tail=e_tail, fwd=e_fwd, out=e_out, mid=e_mid, fin=e_fin, out3=e_out3)
    assert max(e_tail, e_fwd, e_mid, e_fin) <= STATE_TOL
    assert max(e_out, e_out3) <= OUTPUT_TOL
