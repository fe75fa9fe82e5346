"""The calls whose speed matters to a user of this package, as measurable cases.

Each case is one public call: the decode step, the tail replay, the tail
replay continued over a new suffix, the chunked forward (a prompt prefilled
from the zero state, or tokens that continue from a given state) and the whole
linear-attention layer.  Head layouts, lengths and gate ranges are those of the
package's workloads and tests (16 key and 32 value heads of 128 in bf16 for a
hybrid model's layer, 4 heads of 64 in fp32 for the small one).
"""
import math
import random

import torch
import torch.nn.functional as F

import paper_2608_30310_amd as gdn

DEVICE = "cuda:0"
HYBRID = dict(hk=16, hv=32, dk=128, dv=128, dtype="bf16")
SMALL = dict(hk=4, hv=4, dk=64, dv=64, dtype="f32")


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # one token of one conversation: the smallest call, all latency
        dict(HYBRID, name="decode_1", kind="decode", n=1, gate=0.1),
        # one token for every conversation of a serving batch
        dict(HYBRID, name="decode_128", kind="decode", n=128, gate=0.1),
        # a cache hit on a small fp32 layer (2048 tokens matched, 10 % replayed)
        dict(SMALL, name="hit_small_f32", kind="hits", n=1, tail=205, tail_max=205, suffix=256,
             suffix_max=256, lens=0, gate=0.1),
        # a cache hit on one hybrid layer: 8192 tokens matched, 10 % replayed, a question follows
        dict(HYBRID, name="hit_8k", kind="hits", n=1, tail=819, tail_max=819, suffix=512,
             suffix_max=512, lens=0, gate=0.1),
        # the same at 32768 matched tokens
        dict(HYBRID, name="hit_32k", kind="hits", n=1, tail=3277, tail_max=3277, suffix=1024,
             suffix_max=1024, lens=0, gate=0.1),
        # the state alone (5 % of 32768 tokens), as where nothing after it is needed yet
        dict(HYBRID, name="rebuild_1638", kind="tail", n=1, tail=1638, tail_max=1638, lens=0, gate=0.02),
        # 16 concurrent hits of one layer, ragged tails and suffixes
        dict(HYBRID, name="hits_16_ragged", kind="hits", n=16, tail=410, tail_max=3277, suffix=128,
             suffix_max=2048, lens=3, gate=0.1),
        # the same depth of 12 layer groups that replay independently of each other
        dict(HYBRID, name="groups_12", kind="hits", n=12, tail=3277, tail_max=3277, suffix=1024,
             suffix_max=1024, lens=0, gate=0.1),
        # a cache miss: the prompt goes through the chunked forward from the zero state
        dict(HYBRID, name="prefill_8k", kind="forward", n=1, tokens=8192, tokens_max=8192, lens=0,
             from_state=False, gate=0.1),
        # the longest prompt that the package's benchmark knows
        dict(HYBRID, name="prefill_32k", kind="forward", n=1, tokens=32768, tokens_max=32768, lens=0,
             from_state=False, gate=0.02),
        # a whole layer replayed from its cached hiddens, with the output the next layer reads
        dict(HYBRID, name="layer_819", kind="layer", hidden=2048, n=1, tokens=819, tokens_max=819, lens=0,
             outputs=True, act="bf16"),
        # the last layer of a group, of which only the state is needed, in fp32 intermediates
        dict(HYBRID, name="layer_state_3277", kind="layer", hidden=2048, n=1, tokens=3277, tokens_max=3277,
             lens=0, outputs=False, act="f32"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    heads = rng.choice([HYBRID, HYBRID, HYBRID, HYBRID, dict(HYBRID, hk=8, hv=16), dict(HYBRID, dk=64, dv=64),
                        dict(HYBRID, dv=64), dict(HYBRID, dtype="f32"), SMALL])
    gate = rng.choice([0.02, 0.1, 0.5])
    lens = rng.randrange(1 << 20)
    kind = rng.choice(["decode", "hits", "hits", "batch", "batch", "tail", "forward", "forward", "layer"])
    if kind == "decode":
        return dict(heads, kind="decode", n=_log_int(rng, 1, 128), gate=gate)
    part = 2 if heads["dtype"] == "f32" else 1      # fp32 tokens take about twice as long as bf16 ones
    if kind == "hits":
        tail, suffix = _log_int(rng, 100, 3277), _log_int(rng, 32, 2048)
        return dict(heads, kind="hits", n=1, tail=tail, tail_max=tail, suffix=suffix, suffix_max=suffix,
                    lens=lens, gate=gate)
    if kind == "batch":
        # ragged hits; at most as many tokens in all as groups_12
        n = rng.randint(2, 24)
        top = min(3277, 39324 // n) // part
        tail, suffix = _log_int(rng, 64, top), _log_int(rng, 32, min(1024, 12288 // n) // part)
        return dict(heads, kind="hits", n=n, tail=min(tail, 410), tail_max=max(tail, 410), suffix=min(suffix, 128),
                    suffix_max=max(suffix, 128), lens=lens, gate=gate)
    if kind == "tail":
        n = _log_int(rng, 1, 12)
        tail = _log_int(rng, 64, 3277)
        return dict(heads, kind="tail", n=n, tail=max(1, tail // 2), tail_max=tail, lens=lens, gate=gate)
    if kind == "forward":
        n = rng.choice([1, 1, 2, 5])
        top = _log_int(rng, 200, 32768 // n // part)
        return dict(heads, kind="forward", n=n, tokens=max(1, top // 2) if n > 1 else top, tokens_max=top, lens=lens,
                    from_state=rng.random() < 0.5, gate=gate)
    # at most as many multiplications as layer_state_3277
    outputs, act = rng.random() < 0.5, rng.choice(["bf16", "f32"])
    top = _log_int(rng, 64, 1200 if outputs else 3277)
    return dict(HYBRID, kind="layer", hidden=2048, n=1, tokens=top, tokens_max=top, lens=lens, outputs=outputs,
                act=act)


def _lengths(case, name):
    """The lengths of a batch's sequences: `n` of them between the two bounds, by the case alone."""
    lo, hi = case[name], case[name + "_max"]
    rng = random.Random("%d %s" % (case["lens"], name))
    return [hi if lo == hi else rng.randint(lo, hi) for _ in range(case["n"])]


# ------------------------------------------------------------------ inputs
def _offsets(lens):
    cu = torch.zeros(len(lens) + 1, dtype=torch.int32)
    cu[1:] = torch.cumsum(torch.tensor(lens, dtype=torch.int64), 0).to(torch.int32)
    return cu.to(DEVICE), cu


def _tokens(case, lens, gen):
    """q, k, v, g, beta of packed sequences: unit q and k, log gates in (-inf, 0], beta in (0, 1)."""
    T = sum(lens)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    rn = lambda *s: torch.randn(*s, device=DEVICE, generator=gen)
    unit = lambda x: (x / x.norm(dim=-1, keepdim=True)).to(dt)
    cu, cu_host = _offsets(lens)
    return dict(q=unit(rn(T, case["hk"], case["dk"])), k=unit(rn(T, case["hk"], case["dk"])),
                v=rn(T, case["hv"], case["dv"]).to(dt),
                g=(-F.softplus(rn(T, case["hv"])) * case["gate"]).contiguous(),
                beta=torch.sigmoid(rn(T, case["hv"])).contiguous(), cu=cu, cu_host=cu_host)


def _states(case, gen=None):
    """A state per sequence and value head, as large as a rebuilt one; without a generator an empty buffer."""
    shape = (case["n"], case["hv"], case["dk"], case["dv"])
    if gen is None:
        return torch.empty(shape, dtype=torch.float32, device=DEVICE)
    return torch.randn(shape, device=DEVICE, generator=gen) * (2.0 / math.sqrt(case["dk"]))


def _outputs(case, T):
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    return torch.empty((T, case["hv"], case["dv"]), dtype=dt, device=DEVICE)


def _weights(case, gen):
    """One layer's weights in the ranges such layers are initialised with."""
    D, hk, hv, dk, dv = (case[x] for x in ("hidden", "hk", "hv", "dk", "dv"))
    cq, cv = hk * dk, hv * dv
    rn = lambda *s: torch.randn(*s, device=DEVICE, generator=gen)
    ru = lambda *s: torch.rand(*s, device=DEVICE, generator=gen)
    dt = torch.exp(math.log(1e-3) + ru(hv) * math.log(100.0))
    return dict(w_in=(rn(2 * cq + 2 * cv + 2 * hv, D) / D ** 0.5).to(torch.bfloat16), conv_w=ru(2 * cq + cv, 4) - 0.5,
                a_log=torch.log(1 + 15 * ru(hv)), dt_bias=dt + torch.log(-torch.expm1(-dt)), norm_w=0.5 + ru(dv),
                w_out=(rn(D, cv) / cv ** 0.5).to(torch.bfloat16))


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    kind = case["kind"]
    st = dict(case=case)
    if kind == "decode":
        x = _tokens(case, [1] * case["n"], gen)
        st.update(x=x, state_in=_states(case, gen), state_out=_states(case), o=_outputs(case, case["n"]))
    elif kind == "tail":
        st.update(x=_tokens(case, _lengths(case, "tail"), gen), state_out=_states(case))
    elif kind == "forward":
        lens = _lengths(case, "tokens")
        st.update(x=_tokens(case, lens, gen), state_in=_states(case, gen) if case["from_state"] else None,
                  state_out=_states(case), o=_outputs(case, sum(lens)))
    elif kind == "hits":
        suffix = _lengths(case, "suffix")
        st.update(tail=_tokens(case, _lengths(case, "tail"), gen), x=_tokens(case, suffix, gen),
                  state_mid=_states(case), state_out=_states(case), o=_outputs(case, sum(suffix)))
    else:
        lens = _lengths(case, "tokens")
        cu, cu_host = _offsets(lens)
        x = torch.randn(sum(lens), case["hidden"], device=DEVICE, generator=gen).to(torch.bfloat16)
        st.update(x=x, cu=cu, cu_host=cu_host, w=_weights(case, gen), state_out=_states(case),
                  out=torch.empty_like(x) if case["outputs"] else None)
    return st


# ------------------------------------------------------------------ the calls
def run(st):
    case = st["case"]
    kind, x = case["kind"], st["x"]
    if kind == "decode":
        o, s = gdn.decode_step(x["q"], x["k"], x["v"], x["g"], x["beta"], state_in=st["state_in"], o=st["o"],
                               state_out=st["state_out"])
        return dict(o=o, state=s)
    if kind == "tail":
        return dict(state=gdn.tail_replay(x["k"], x["v"], x["g"], x["beta"], x["cu"], x["cu_host"],
                                          state_out=st["state_out"]))
    if kind == "forward":
        o, s = gdn.chunk_forward(x["q"], x["k"], x["v"], x["g"], x["beta"], x["cu"], x["cu_host"],
                                 state_in=st["state_in"], o=st["o"], state_out=st["state_out"])
        return dict(o=o, state=s)
    if kind == "hits":
        t = st["tail"]
        o, mid, s = gdn.replay_forward(t["k"], t["v"], t["g"], t["beta"], t["cu"], x["q"], x["k"], x["v"], x["g"],
                                       x["beta"], x["cu"], cu_tail_host=t["cu_host"], cu_suf_host=x["cu_host"],
                                       state_mid=st["state_mid"], o=st["o"], state_out=st["state_out"])
        return dict(o=o, rebuilt=mid, state=s)
    s, out = gdn.la_block_replay(x, st["w"], st["cu"], case["hk"], case["hv"], case["dk"], case["dv"],
                                 case["dk"] ** -0.5, cu_seqlens_host=st["cu_host"], outputs=case["outputs"],
                                 act_dtype=case["act"], state_out=st["state_out"], out=st["out"])
    return dict(state=s, out=out) if case["outputs"] else dict(state=s)


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    """Each input read once, each output written once; the recurrence token by token: per token and value head
    two products with the state (recall and write), three where there are outputs."""
    kind, n, hk, hv, dk, dv = (case[x] for x in ("kind", "n", "hk", "hv", "dk", "dv"))
    es = 2 if case["dtype"] == "bf16" else 4
    state = n * hv * dk * dv * 4
    kv = hk * dk * es + hv * dv * es + hv * 8            # k, v, g, beta of a token
    qo = hk * dk * es + hv * dv * es                     # q, o
    one = 2 * hv * dk * dv                               # one product with the state
    if kind == "decode":
        return dict(bytes=2 * state + n * (kv + qo), flops=3 * one * n)
    if kind == "tail":
        T = sum(_lengths(case, "tail"))
        return dict(bytes=T * kv + state, flops=2 * one * T)
    if kind == "forward":
        T = sum(_lengths(case, "tokens"))
        return dict(bytes=T * (kv + qo) + state * (2 if case["from_state"] else 1), flops=3 * one * T)
    if kind == "hits":
        T, S = sum(_lengths(case, "tail")), sum(_lengths(case, "suffix"))
        return dict(bytes=T * kv + S * (kv + qo) + 2 * state, flops=2 * one * T + 3 * one * S)
    T, D = sum(_lengths(case, "tokens")), case["hidden"]
    cq, cv = hk * dk, hv * dv
    if case["outputs"]:
        rows = 2 * cq + 2 * cv + 2 * hv
        return dict(bytes=2 * D * (rows + cv) + T * 4 * D + state, flops=2 * T * D * (rows + cv) + 3 * one * T)
    rows = cq + cv + 2 * hv
    return dict(bytes=2 * D * rows + T * 2 * D + state, flops=2 * T * D * rows + 2 * one * T)


def tolerance(case):
    """About four times the error against 64 bits that the calls show: bf16 outputs are off by their rounding
    (1.7e-3), states of bf16 tokens by the products' (up to 5e-4), fp32 ones by the split operands' (5e-6); a layer
    with bf16 intermediates by theirs (5e-3)."""
    if case["kind"] == "layer":
        if case["act"] == "bf16":
            return dict(rel=2e-2)
        return dict(rel=8e-3) if case["outputs"] else dict(rel=4e-5)
    if case["dtype"] == "f32":
        return dict(rel=4e-6 if case["kind"] == "decode" else 2e-5)
    return dict(rel=2e-3) if case["kind"] == "tail" else dict(rel=7e-3)


# ------------------------------------------------------------------ the same in 64 bits
def _recurrence(x, n, state, outputs):
    """Token by token in fp64, every sequence and value head at once: with M the state (d_k x d_v),
    M <- e^g M; M <- M + k (beta (v - M^T k))^T; o = M^T q.  Shorter sequences are padded with tokens that
    leave the state alone (g = beta = 0).  x: q, k, v, g, beta [T, ...] and the host offsets."""
    cu = x["cu_host"].tolist()
    lens = [cu[i + 1] - cu[i] for i in range(n)]
    L = max(lens)
    v = x["v"]
    hv, dv = v.shape[1:]
    hk, dk = x["k"].shape[1:]

    def padded(t):
        p = torch.zeros((L, n) + tuple(t.shape[1:]), dtype=torch.float64, device=t.device)
        for i in range(n):
            p[:lens[i], i] = t[cu[i]:cu[i + 1]].double()
        return p

    heads = lambda t: t.repeat_interleave(hv // hk, dim=1)      # value head h reads key head h // (hv // hk)
    k, vv = padded(x["k"]), padded(v)
    q = padded(x["q"]) if outputs else None
    alpha, beta = torch.exp(padded(x["g"])), padded(x["beta"])
    M = torch.zeros((n, hv, dk, dv), dtype=torch.float64, device=v.device) if state is None else state.double().clone()
    o = torch.zeros((sum(lens), hv, dv), dtype=torch.float64, device=v.device) if outputs else None
    os = torch.empty((L, n, hv, dv), dtype=torch.float64, device=v.device) if outputs else None
    for t in range(L):
        kt = heads(k[t])
        M *= alpha[t][:, :, None, None]
        u = torch.matmul(kt.unsqueeze(2), M).squeeze(2)
        d = beta[t].unsqueeze(2) * (vv[t] - u)
        M.addcmul_(kt.unsqueeze(3), d.unsqueeze(2))
        if outputs:
            os[t] = torch.matmul(heads(q[t]).unsqueeze(2), M).squeeze(2)
    if outputs:
        for i in range(n):
            o[cu[i]:cu[i + 1]] = os[:lens[i], i]
    return o, M


def _layer(case, st):
    """The layer in fp64: projection, causal 4-tap convolution per sequence, SiLU, unit q and k, the gates, the
    recurrence from zero, the gated RMS norm and the output projection."""
    hk, hv, dk, dv = (case[x] for x in ("hk", "hv", "dk", "dv"))
    cq, cv, n = hk * dk, hv * dv, case["n"]
    w = {name: t.double() for name, t in st["w"].items()}
    P = st["x"].double() @ w["w_in"].t().contiguous()
    T = P.shape[0]
    cu = st["cu_host"].tolist()
    c = torch.zeros((T, 2 * cq + cv), dtype=torch.float64, device=P.device)
    for i in range(n):
        a, b = cu[i], cu[i + 1]
        for j in range(4):
            s = 3 - j
            if b - a > s:
                c[a + s:b] += P[a:b - s, :2 * cq + cv] * w["conv_w"][:, j]
    c = c * torch.sigmoid(c)
    unit = lambda t: t / torch.sqrt((t * t).sum(-1, keepdim=True) + 1e-6)
    at = 2 * cq + cv
    x = dict(q=unit(c[:, :cq].reshape(T, hk, dk)), k=unit(c[:, cq:2 * cq].reshape(T, hk, dk)),
             v=c[:, 2 * cq:].reshape(T, hv, dv).contiguous(),
             g=-torch.exp(w["a_log"]) * F.softplus(P[:, at:at + hv] + w["dt_bias"]),
             beta=torch.sigmoid(P[:, at + hv:at + 2 * hv]), cu_host=st["cu_host"])
    o, M = _recurrence(x, n, None, case["outputs"])
    if not case["outputs"]:
        return dict(state=M)
    o = o * dk ** -0.5
    z = P[:, at + 2 * hv:].reshape(T, hv, dv)
    y = o / torch.sqrt((o * o).mean(-1, keepdim=True) + 1e-6) * w["norm_w"] * z * torch.sigmoid(z)
    return dict(state=M, out=y.reshape(T, cv) @ w["w_out"].t().contiguous())


def exact(case, seed):
    st = prepare(case, seed)
    kind = case["kind"]
    if kind == "layer":
        return _layer(case, st)
    x, n = st["x"], case["n"]
    if kind == "decode":
        o, s = _recurrence(dict(x, cu_host=torch.arange(n + 1)), n, st["state_in"], True)
        return dict(o=o, state=s)
    if kind == "tail":
        return dict(state=_recurrence(x, n, None, False)[1])
    if kind == "forward":
        o, s = _recurrence(x, n, st["state_in"], True)
        return dict(o=o, state=s)
    _, mid = _recurrence(st["tail"], n, None, False)
    o, s = _recurrence(x, n, mid, True)
    return dict(o=o, rebuilt=mid, state=s)
