"""Performance cases of the decoder: the calls a program makes through
``paper_2211_00484_amd.tbs``, over the range of sizes it makes them at.

listed()  the named cases; draw(rng) gives more of the same ranges.
prepare(case, seed)  model, graph and inputs on the GPU; run(state) one pass.
work(case)  bytes and operations a pass cannot do without.
exact(case, seed)  the same outputs in 64 bits, in plain torch.

Inputs are shaped like those of a trained model rather than flat noise: every encoder
frame leans towards the joiner row of a target symbol (blank on about three frames of
four, and otherwise the next label of a random sequence, walked along the decoding graph
where there is one), confidently on most frames and ambiguously on some, plus unit noise.
"""
import functools
import math

import numpy as np
import torch

from paper_2211_00484_amd import synth, tbs

DEV = "cuda"


# ---------------------------------------------------------------------------
# the cases

def _decode(name, B, T, lo, C, V, dtype, graph, beam, Ns, Nc, **more):
    c = dict(kind="decode", B=B, T=T, lo=lo, C=C, V=V, dtype=dtype, graph=graph, beam=beam,
             states=Ns, contexts=Nc, **more)
    return dict(c, name=name) if name else c


INF = 1e30  # "no beam" as a plain number


def listed():
    return [
        # one short utterance pair on a toy model: launch latency and the host path
        _decode("tiny", 2, 20, 20, 32, 16, "fp32", "trivial", INF, 4, 4),
        # the benchmark's default: a batch of 4 to 10 s utterances, 500 word pieces, beam 4
        _decode("standard", 32, 250, 100, 512, 500, "fp32", "trivial", INF, 4, 4),
        # the same batch constrained by a 5,000-state decoding graph
        _decode("graph", 32, 250, 100, 512, 500, "fp32", "uniform", 4.0, 32, 8,
                graph_states=5000, graph_arcs=100_000),
        # offline transcription at full batch with 16-bit joiner operands
        _decode("throughput", 256, 250, 250, 512, 500, "bf16", "trivial", INF, 4, 4),
        # large vocabulary and a large lexicon-like graph, in both joiner precisions
        _decode("large", 128, 500, 300, 512, 5000, "fp32", "powerlaw", 8.0, 64, 16,
                graph_states=1_000_000, graph_arcs=5_000_000),
        _decode("large_bf16", 128, 500, 300, 512, 5000, "bf16", "powerlaw", 8.0, 64, 16,
                graph_states=1_000_000, graph_arcs=5_000_000),
        # live captions: the standard batch fed in chunks of 0.64 s
        dict(_decode("streaming", 32, 250, 100, 512, 500, "fp32", "trivial", INF, 4, 4),
             kind="chunks", chunk=16),
        # the best label sequence by total probability: lattice and 100 sampled paths
        dict(_decode("logadd", 32, 250, 100, 512, 500, "fp32", "trivial", INF, 4, 4),
             kind="logadd", paths=100),
        # the comparison search over whole label sequences
        dict(name="hyps", kind="hyps", B=32, T=250, lo=100, C=512, V=500, dtype="fp32",
             beam_size=4, merge="logadd"),
        # rescoring: joiner log-probabilities of given (frame, context) pairs
        dict(name="joiner_rows", kind="joiner", R=6000, C=512, V=500, dtype="fp32"),
        # loss forward of a training batch of 10 s utterances (all cells kept, for a backward)
        dict(name="loss_modified", kind="transducer", form="modified", B=32, T=250, lo=250,
             U=80, ulo=40, alpha=True),
        # likelihoods of a large scoring batch of ragged utterances
        dict(name="loss_standard", kind="transducer", form="standard", B=1024, T=250, lo=125,
             U=80, ulo=40, alpha=False),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(["decode", "decode", "decode", "decode", "chunks", "logadd", "hyps",
                           "joiner", "transducer"])
        if kind == "transducer":
            T, U = _logint(rng, 40, 600), _logint(rng, 8, 200)
            T = max(T, U + 1)  # a label moves to the next frame: no fewer frames than labels
            alpha = rng.random() < 0.5
            c = dict(kind=kind, form=rng.choice(["standard", "modified", "constrained"]),
                     B=_logint(rng, 1, 1024), T=T,
                     lo=T if alpha else max(U, T // 2), U=U, ulo=U // 2, alpha=alpha)
            if c["B"] * T * U <= 40_000_000:
                return c
            continue
        V = _logint(rng, 16, 5000)
        C = rng.choice([rng.randint(32, 768), 256, 512, 640])
        dtype = rng.choice(["fp32", "bf16"])
        if kind == "joiner":
            c = dict(kind=kind, R=_logint(rng, 16, 16000), C=C, V=V, dtype=dtype)
            if c["R"] * V <= 40_000_000:
                return c
            continue
        B, T = _logint(rng, 1, 256), _logint(rng, 16, 400)
        lo = rng.choice([T, max(1, T // 2), max(1, T // 4)])
        if kind == "hyps":
            c = dict(kind=kind, B=min(B, 64), T=min(T, 250), lo=min(lo, 250), C=C, V=V,
                     dtype=dtype, beam_size=rng.randint(1, 8),
                     merge=rng.choice(["max", "logadd"]))
            if c["B"] * c["T"] * V * c["beam_size"] * C <= 1.0e12:
                return c
            continue
        graph = rng.choice(["trivial", "uniform", "powerlaw"])
        if kind == "logadd":
            graph = rng.choice(["trivial", "uniform"])
        if graph == "trivial":
            Ns = rng.randint(2, 12)
            c = _decode(None, B, T, lo, C, V, dtype, graph, INF, Ns, rng.randint(2, Ns))
        else:
            Ns = _logint(rng, 4, 64)
            S = _logint(rng, 100, 200_000 if graph == "powerlaw" else 20_000)
            c = _decode(None, B, T, lo, C, V, dtype, graph, rng.choice([4.0, 6.0, 8.0]), Ns,
                        rng.randint(2, min(Ns, 16)), graph_states=S,
                        graph_arcs=S * rng.randint(3, 20))
            if kind == "decode" and rng.random() < 0.25:
                c["graphs"] = 2  # two graphs alternating over the streams
        rows = c["B"] * c["contexts"]
        if rows * T * V * C > 1.2e12:
            continue
        if kind == "chunks":
            c = dict(c, kind=kind, chunk=_logint(rng, 4, 64))
        if kind == "logadd":
            c = dict(c, kind=kind, B=min(B, 64), T=min(T, 250), lo=min(lo, 250), states=min(Ns, 32),
                     contexts=min(c["contexts"], 32, Ns), paths=_logint(rng, 20, 200))
        return c


# ---------------------------------------------------------------------------
# inputs

@functools.lru_cache(maxsize=6)
def _host_graph(kind, S, A, V, which):
    """The decoding graph of a deployment, on the host; the same for every seed, as a
    program keeps one graph for all its inputs."""
    if kind == "trivial":
        return synth.trivial_graph(V)
    if kind == "uniform":
        return synth.uniform_random_graph(S, A, V, seed=1 + which)
    return synth.power_law_graph(S, A, V, seed=1 + which)


def _graphs(c):
    n = c.get("graphs", 1)
    return [_host_graph(c.get("graph", "trivial"), c.get("graph_states", 1),
                        c.get("graph_arcs", 0), c["V"], i) for i in range(n)]


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _weights(c, g):
    """Embedding, conv taps, joiner weight and bias, float32."""
    V, C = c["V"], c["C"]

    def n(*s):
        return torch.randn(*s, generator=g, device=DEV)

    return dict(E=n(V, C), conv=0.4 * n(C, 2), W=(0.05 * math.sqrt(512 / C)) * n(V, C),
                b=0.05 * n(V))


def _lengths(c, rng):
    lens = rng.integers(c["lo"], c["T"] + 1, size=c["B"]).astype(np.int32)
    lens[int(rng.integers(0, c["B"]))] = c["T"]
    return lens


def _targets(c, rng, graphs):
    """Target symbol of every frame, [B, T] (0 = blank)."""
    B, T, V = c["B"], c["T"], c["V"]
    emit = rng.random((B, T)) < 0.25
    if c.get("graph", "trivial") == "trivial":
        return np.where(emit, rng.integers(1, V, size=(B, T)), 0)
    out = np.zeros((B, T), np.int64)
    pick = rng.random((B, T))
    for k, g in enumerate(graphs):  # a random walk along each stream's graph
        rows = np.arange(k, B, len(graphs))
        st = np.full(len(rows), g.start)
        for t in range(T):
            lo, deg = g.row_ptr[st], g.row_ptr[st + 1] - g.row_ptr[st]
            on = emit[rows, t] & (deg > 0)
            a = np.where(on, lo + (pick[rows, t] * deg).astype(np.int64), 0)
            out[rows, t] = np.where(on, g.label[a], 0)
            st = np.where(on, g.dest[a], st)
    return out


def _encoder(c, g, w, targets):
    B, T = targets.shape
    clear = 0.4 + 0.8 * torch.rand(B, T, 1, generator=g, device=DEV)
    vague = 0.1 + 0.4 * torch.rand(B, T, 1, generator=g, device=DEV)
    lean = torch.where(torch.rand(B, T, 1, generator=g, device=DEV) < 0.7, clear, vague)
    enc = torch.randn(B, T, c["C"], generator=g, device=DEV)
    Wn = w["W"] / w["W"].square().mean().sqrt()
    enc += lean * Wn[torch.from_numpy(targets).to(DEV)]
    return enc


def _inputs(case, seed):
    """Everything a pass needs, as plain tensors and arrays (before any handle)."""
    c, g = case, _gen(seed)
    rng = np.random.default_rng(int(seed))
    if c["kind"] == "transducer":
        B, T, U = c["B"], c["T"], c["U"]
        x = 2.0 * torch.randn(B, T, U + 1, generator=g, device=DEV)
        blank = torch.nn.functional.logsigmoid(x)
        label = torch.nn.functional.logsigmoid(-x[:, :, :U]) - 0.3 * torch.rand(
            B, T, U, generator=g, device=DEV)
        lens = np.stack([_lengths(c, rng), rng.integers(c["ulo"], U + 1, size=B)], 1)
        return dict(blank=blank.contiguous(), label=label.contiguous(),
                    lens=torch.from_numpy(lens.astype(np.int32)).to(DEV))
    w = _weights(c, g)
    if c["kind"] == "joiner":
        R, V = c["R"], c["V"]
        ctx = torch.from_numpy((rng.integers(0, V, R) * V + rng.integers(0, V, R)).astype(np.int32))
        tgt = rng.integers(0, V, size=(1, R))
        return dict(w=w, ctx=ctx.to(DEV), enc=_encoder(c, g, w, tgt)[0].contiguous())
    graphs = _graphs(c)
    lens = _lengths(c, rng)
    enc = _encoder(c, g, w, _targets(c, rng, graphs))
    x = dict(w=w, enc=enc, lens=lens, graphs=graphs)
    if c["kind"] == "logadd":
        x["uniforms"] = torch.rand(c["B"], c["paths"], c["T"] + 1, generator=g, device=DEV,
                                   dtype=torch.float64)
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    st = dict(x, case=case)
    if case["kind"] == "transducer":
        return st
    w = x["w"]
    st["model"] = tbs.Model(case["V"], case["C"], w["E"], w["conv"], w["W"], w["b"],
                            dtype=case["dtype"])
    del st["w"]
    if "graphs" in x:
        gs = [tbs.Graph.trivial(case["V"]) if case.get("graph", "trivial") == "trivial"
              else tbs.Graph.from_synth(g) for g in x["graphs"]]
        st["graph"] = gs[0] if len(gs) == 1 else [gs[i % len(gs)] for i in range(case["B"])]
    if case["kind"] == "chunks":  # the frames arrive chunk by chunk
        n = case["chunk"]
        st["chunks"] = [(st["enc"][:, i:i + n].contiguous(), np.clip(st["lens"] - i, 0, n).astype(np.int32))
                        for i in range(0, case["T"], n)]
        del st["enc"]
    return st


# ---------------------------------------------------------------------------
# one pass

def _beam(c):
    return math.inf if c["beam"] >= INF else c["beam"]


def _decoded(out):
    return dict(tokens=out.tokens, num_tokens=out.num_tokens, scores=out.scores,
                status=out.status)


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "decode":
        return _decoded(tbs.decode(s["model"], s["graph"], s["enc"], s["lens"], beam=_beam(c),
                                   max_states=c["states"], max_contexts=c["contexts"]))
    if kind == "chunks":
        ds = tbs.DecodeState(s["model"], s["graph"], c["B"], c["T"], beam=_beam(c),
                             max_states=c["states"], max_contexts=c["contexts"])
        for enc, lens in s["chunks"]:
            ds.chunk(enc, lens)
        out = ds.finish()
        ds.close()
        return _decoded(out)
    if kind == "logadd":
        lat = tbs.Lattice(s["model"], s["graph"], s["enc"], s["lens"], beam=_beam(c),
                          max_states=c["states"], max_contexts=c["contexts"])
        out = lat.nbest(c["paths"], s["uniforms"])
        lat.close()
        return dict(tokens=out.tokens, num_tokens=out.num_tokens, scores=out.scores)
    if kind == "hyps":
        out = tbs.hyp_search(s["model"], s["enc"], s["lens"], beam_size=c["beam_size"],
                             merge=c["merge"])
        return dict(tokens=out.tokens, num_tokens=out.num_tokens, scores=out.scores)
    if kind == "joiner":
        return dict(logp=tbs.joiner_logp(s["model"], s["enc"], s["ctx"]))
    total, alpha, status = tbs.transducer_forward(c["form"], s["blank"], s["label"], s["lens"],
                                                  want_alpha=c["alpha"])
    out = dict(total=total, status=status)
    if c["alpha"]:  # eq. (1) visits rows 0 .. T - 1, eq. (2) and (3) rows 0 .. T
        out["alpha"] = alpha[:, :c["T"]] if c["form"] == "standard" else alpha
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how far another correct one may be

def work(case):
    c = case
    if c["kind"] == "transducer":
        B = c["B"]
        T, U = (c["T"] + c["lo"]) / 2, (c["U"] + c["ulo"]) / 2
        cells = B * T * (2 * U + 1)
        return {"bytes": 4 * cells + (4 * B * (T + 1) * (c["U"] + 1) if c["alpha"] else 0) + 20 * B,
                "flops": 6 * B * T * (U + 1)}
    V, C = c["V"], c["C"]
    wbytes = V * C * (4 if c["dtype"] == "fp32" else 2)
    if c["kind"] == "joiner":
        R = c["R"]
        return {"bytes": wbytes + 4 * R * (C + V + 1) + 8 * min(R, V) * C, "flops": 2 * R * V * C}
    frames = c["B"] * (c["T"] + c["lo"]) / 2
    rows = c["beam_size"] if c["kind"] == "hyps" else c["contexts"]
    if c.get("beam", INF) < INF:
        rows = max(1, rows // 2)  # a beam leaves about half of the contexts it may
    return {"bytes": wbytes + 4 * frames * C + 4 * c["B"] * (c["T"] + 4),
            "flops": 2 * frames * rows * V * C}


def tolerance(case):
    c = case
    if c["kind"] == "transducer":  # fp64 totals; alpha rounded to fp32
        return {"rel": 2e-7, "max": 1e-6}
    if c["kind"] == "joiner":
        # fp32: sums of C products and the log-softmax; bf16: a tanh that rounds to the
        # neighbouring bf16 value
        return {"rel": 4e-7, "max": 4e-6} if c["dtype"] == "fp32" else {"rel": 5e-5, "max": 1e-3}
    # path scores; a near-tie that falls the other way moves a stream's tokens
    return ({"rel": 1e-6, "max": 1e-5, "differ": 0.01} if c["dtype"] == "fp32"
            else {"rel": 1e-5, "max": 1e-4, "differ": 0.01})


# ---------------------------------------------------------------------------
# the same in 64 bits

NEG = -math.inf


def _logp64(c, w, enc, ctx):
    """log P(. | ctx, frame): enc [R, C], ctx [R] -> [R, V] float64."""
    V = c["V"]
    E, conv, W, b = (w[k].double() for k in ("E", "conv", "W", "b"))
    dec = torch.relu(conv[:, 0] * E[ctx // V] + conv[:, 1] * E[ctx % V])
    h = torch.tanh(enc.double() + dec)
    if c["dtype"] == "bf16":
        h, W = h.to(torch.bfloat16).double(), w["W"].to(torch.bfloat16).double()
    return torch.log_softmax(h @ W.t() + b, -1)


def _csr(graphs, B):
    """The streams' graphs side by side: CSR tensors and each stream's start state."""
    rp, dest, label, q, start, base, off = [], [], [], [], [], 0, 0
    for g in graphs:
        rp.append(g.row_ptr[:-1].astype(np.int64) + off)
        dest.append(g.dest.astype(np.int64) + base)
        label.append(g.label.astype(np.int64))
        q.append(g.score.astype(np.float64))
        start.append(g.start + base)
        base += g.num_states
        off += g.num_arcs
    rp.append(np.array([off]))

    def t(a):
        return torch.from_numpy(np.concatenate(a)).to(DEV)

    starts = torch.tensor([start[b % len(graphs)] for b in range(B)], device=DEV)
    return t(rp), t(dest), t(label), t(q), starts, base


def _search64(c, x, visit=None):
    """Beam search in float64; returns the best final scores [B].  visit(t, active, before,
    after, lp): the survivors (ctx, state, score, valid), [B, Ns] each, around frame t."""
    B, T, V, Ns, Nc = c["B"], c["T"], c["V"], c["states"], min(c["contexts"], c["states"])
    rp, dest, label, q, starts, S = _csr(x["graphs"], B)
    lens = torch.from_numpy(x["lens"]).to(DEV)
    ctx = torch.zeros(B, Ns, dtype=torch.int64, device=DEV)
    state = starts[:, None].repeat(1, Ns)
    score = torch.full((B, Ns), NEG, dtype=torch.float64, device=DEV)
    score[:, 0] = 0.0
    valid = score > NEG
    bidx = torch.arange(B, device=DEV)[:, None].expand(B, Ns)
    for t in range(T):
        live = valid & (t < lens)[:, None]
        b, i = bidx[live], torch.nonzero(live)[:, 1]
        k0, s0, sc0 = ctx[live], state[live], score[live]
        lp = _logp64(c, x["w"], x["enc"][b, t], k0)
        deg = rp[s0 + 1] - rp[s0]
        src = torch.repeat_interleave(torch.arange(len(b), device=DEV), deg)
        pos = torch.arange(len(src), device=DEV) - (torch.cumsum(deg, 0) - deg)[src]
        a = rp[s0][src] + pos
        cb = torch.cat([b, b[src]])
        ck = torch.cat([k0, (k0[src] % V) * V + label[a]])
        cs = torch.cat([s0, dest[a]])
        cv = torch.cat([sc0 + lp[:, 0], sc0[src] + q[a] + lp[src, label[a]]])
        # drop what is below each stream's beam before the merge, then keep each key's best
        best = torch.full((B,), NEG, dtype=torch.float64, device=DEV).scatter_reduce(0, cb, cv, "amax")
        keep = cv >= best[cb] - _beam(c) if _beam(c) < math.inf else cv > NEG
        if _beam(c) == math.inf and len(cb) > 4 * B * Ns * Ns:
            # no beam: at most Ns kept tuples, each merging candidates of at most Ns parents
            m = torch.full((B, Ns * V), NEG, dtype=torch.float64, device=DEV)
            slot = torch.cat([i * V, i[src] * V + label[a]])
            m[cb, slot] = cv
            kth = m.topk(min(Ns * Ns + 1, Ns * V), 1).values[:, -1]
            keep = cv >= kth[cb]
        cb, ck, cs, cv = cb[keep], ck[keep], cs[keep], cv[keep]
        key = (cb * S + cs) * (V * V) + ck
        order = torch.argsort(cv, descending=True, stable=True)
        order = order[torch.argsort(key[order], stable=True)]
        first = torch.ones(len(order), dtype=torch.bool, device=DEV)
        first[1:] = key[order][1:] != key[order][:-1]
        u = order[first]
        cb, ck, cs, cv = cb[u], ck[u], cs[u], cv[u]
        o = torch.argsort(cv, descending=True, stable=True)
        o = o[torch.argsort(cb[o], stable=True)]
        cb, ck, cs, cv = cb[o], ck[o], cs[o], cv[o]
        at = torch.searchsorted(cb, torch.arange(B, device=DEV))
        rank = torch.arange(len(cb), device=DEV) - at[cb]
        k = rank < Ns
        cb, ck, cs, cv, rank = cb[k], ck[k], cs[k], cv[k], rank[k]
        nk = torch.full((B, Ns), -1, dtype=torch.int64, device=DEV)
        ns, nv = torch.zeros_like(nk), torch.full((B, Ns), NEG, dtype=torch.float64, device=DEV)
        nk[cb, rank], ns[cb, rank], nv[cb, rank] = ck, cs, cv
        # a context's rank: the distinct contexts that appear before its first tuple
        same = nk[:, :, None] == nk[:, None, :]
        lead = same.float().argmax(2)
        isf = (lead == torch.arange(Ns, device=DEV)) & (nv > NEG)
        crank = (torch.cumsum(isf.long(), 1) - isf.long()).gather(1, lead)
        nvalid = (nv > NEG) & (crank < Nc)
        # canonical order: (context, state) ascending, empty slots last
        ck = torch.where(nvalid, nk * S + ns, torch.full_like(nk, 1 << 62))
        o = torch.argsort(ck, 1)
        nk, ns, nv, nvalid = nk.gather(1, o), ns.gather(1, o), nv.gather(1, o), nvalid.gather(1, o)
        act = (t < lens)[:, None]
        if visit is not None:
            full = torch.zeros(B, Ns, V, dtype=torch.float64, device=DEV)
            full[b, i] = lp
            visit(t, act[:, 0], (ctx, state, valid), (nk, ns, nvalid), full)
        ctx, state = torch.where(act, nk, ctx), torch.where(act, ns, state)
        score = torch.where(act, torch.where(nvalid, nv, torch.full_like(nv, NEG)), score)
        valid = torch.where(act, nvalid, valid)
    return score.amax(1)


def _logadd64(c, x):
    """Total log probability of the best of the label sequences sampled from the lattice."""
    B, T, V, Ns, n = c["B"], c["T"], c["V"], c["states"], c["paths"]
    rp, dest, label, q, _, _ = _csr(x["graphs"], B)
    lens = torch.from_numpy(x["lens"]).to(DEV)
    PB, PL, LAB, AL = [], [], [], []  # per frame: blank and label arc weights [B, dst, src]
    al = torch.full((B, Ns), NEG, dtype=torch.float64, device=DEV)
    al[:, 0] = 0.0
    AL.append(al)
    deg = int((rp[1:] - rp[:-1]).max())
    trivial = c["graph"] == "trivial"

    def visit(t, act, before, after, lp):
        (k0, s0, v0), (k1, s1, v1) = before, after
        pair = v1[:, :, None] & v0[:, None, :] & act[:, None, None]
        neg = torch.full((B, Ns, Ns), NEG, dtype=torch.float64, device=DEV)
        stay = pair & (k0[:, None, :] == k1[:, :, None]) & (s0[:, None, :] == s1[:, :, None])
        pb = torch.where(stay, lp[:, None, :, 0].expand(B, Ns, Ns), neg)
        lab = torch.where(v1, k1 % V, torch.zeros_like(k1))
        lpl = lp.gather(2, lab[:, None, :].expand(B, Ns, Ns)).transpose(1, 2)
        move = pair & (k0[:, None, :] % V == torch.div(k1, V, rounding_mode="floor")[:, :, None]) & (lab > 0)[:, :, None]
        if trivial:
            w = torch.zeros_like(lpl)
        else:
            lo, d = rp[s0], rp[s0 + 1] - rp[s0]
            j = torch.arange(deg, device=DEV)
            a = (lo[:, :, None] + torch.minimum(j, (d - 1).clamp(min=0)[:, :, None])).clamp(max=len(dest) - 1)
            ok = j < d[:, :, None]
            hit = (ok[:, None] & (label[a][:, None] == lab[:, :, None, None])
                   & (dest[a][:, None] == s1[:, :, None, None]))
            w = torch.where(hit, q[a][:, None].expand_as(hit), torch.full((), NEG, dtype=torch.float64, device=DEV)).logsumexp(-1)
        pl = torch.where(move, lpl + w, neg)
        PB.append(pb), PL.append(pl), LAB.append(lab)
        prev = AL[-1]
        na = torch.logaddexp(pb + prev[:, None, :], pl + prev[:, None, :]).logsumexp(2)
        AL.append(torch.where(act[:, None], na, prev))

    _search64(c, x, visit)
    # backward sampling by inversion: the final node, then the arc into each node
    u = x["uniforms"]

    def pick(v, uu):
        p = torch.exp(v - v.amax(-1, keepdim=True))
        cum = p.cumsum(-1)
        return (cum > (uu * cum[..., -1])[..., None]).long().argmax(-1)

    ul = u.gather(2, lens.long()[:, None, None].expand(B, n, 1))[:, :, 0]
    node = pick(AL[-1][:, None, :].expand(B, n, Ns), ul)
    bi = torch.arange(B, device=DEV)[:, None].expand(B, n)
    labels = torch.zeros(B, n, T, dtype=torch.int64, device=DEV)
    for f in range(T - 1, -1, -1):
        act = (f < lens)[:, None]
        v = torch.stack([PB[f], PL[f]], -1) + AL[f][:, None, :, None]
        k = pick(v.reshape(B, Ns, 2 * Ns)[bi, node], u[:, :, f])
        labels[:, :, f] = torch.where(act & (k % 2 == 1), LAB[f][bi, node], 0)
        node = torch.where(act, k // 2, node)
    lab = labels.cpu().numpy()
    own, seqs = [], []
    for b in range(B):
        for y in dict.fromkeys(tuple(r[r > 0]) for r in lab[b]):
            own.append(b)
            seqs.append(y)
    K = max(1, max(len(y) for y in seqs))
    Y = torch.zeros(len(seqs), K, dtype=torch.int64)
    for s, y in enumerate(seqs):
        Y[s, :len(y)] = torch.tensor(y, dtype=torch.int64)
    Y, own = Y.to(DEV), torch.tensor(own, device=DEV)
    ny = torch.tensor([len(y) for y in seqs], device=DEV)
    A = torch.zeros(len(seqs), Ns, K + 1, dtype=torch.float64, device=DEV)
    A[:, 0, 0] = 1.0
    scale = torch.zeros(len(seqs), dtype=torch.float64, device=DEV)
    for f in range(T):
        act = (f < lens)[own]
        new = torch.bmm(torch.exp(PB[f])[own].contiguous(), A)
        lab_to = torch.bmm(torch.exp(PL[f])[own].contiguous(), A[:, :, :-1].contiguous())
        new[:, :, 1:] += lab_to * (LAB[f][own][:, :, None] == Y[:, None, :])
        m = new.amax((1, 2))
        m = torch.where(m > 0, m, torch.ones_like(m))
        A = torch.where(act[:, None, None], new / m[:, None, None], A)
        scale = torch.where(act, scale + m.log(), scale)
    tot = A.sum(1).gather(1, ny[:, None])[:, 0].log() + scale
    return torch.full((B,), NEG, dtype=torch.float64, device=DEV).scatter_reduce(0, own, tot, "amax")


def _hyps64(c, x):
    """Best score of the full-sequence beam search, [B]."""
    B, T, V, N = c["B"], c["T"], c["V"], c["beam_size"]
    lens = torch.from_numpy(x["lens"]).to(DEV)
    score = torch.full((B, N), NEG, dtype=torch.float64, device=DEV)
    score[:, 0] = 0.0
    h = torch.full((B, N), 1234567, dtype=torch.int64, device=DEV)
    ph, cnt, ctx = torch.zeros_like(h), torch.zeros_like(h), torch.zeros_like(h)
    for t in range(T):
        lp = _logp64(c, x["w"], x["enc"][:, t].repeat_interleave(N, 0), ctx.reshape(-1)).reshape(B, N, V)
        cand = score[:, :, None] + lp
        # the blank of y_i and label last(y_i) of y_j give the same sequence
        same = (h[:, None, :] == ph[:, :, None]) & (cnt[:, None, :] == cnt[:, :, None] - 1)
        same &= (score > NEG)[:, :, None] & (score > NEG)[:, None, :]
        hit, j = same.any(2), same.long().argmax(2)
        last = ctx % V
        bb = torch.arange(B, device=DEV)[:, None].expand(B, N)
        other = torch.where(hit, cand[bb, j, last], torch.full_like(score, NEG))
        blank = cand[:, :, 0]
        merged = torch.logaddexp(blank, other) if c["merge"] == "logadd" else torch.maximum(blank, other)
        cand[bb[hit], j[hit], last[hit]] = NEG
        cand[:, :, 0] = merged
        top = cand.reshape(B, N * V).topk(min(N, N * V), 1)
        i, k = top.indices // V, top.indices % V
        lab = k > 0
        hi, pi, ci, xi = (v.gather(1, i) for v in (h, ph, cnt, ctx))
        act = (t < lens)[:, None]
        score = torch.where(act, top.values, score)
        ph = torch.where(act, torch.where(lab, hi, pi), ph)
        cnt = torch.where(act, torch.where(lab, ci + 1, ci), cnt)
        ctx = torch.where(act, torch.where(lab, xi % V * V + k, xi), ctx)
        h = torch.where(act, torch.where(lab, hi * 6364136223846793005 + k, hi), h)
    return score.amax(1)


def _transducer64(c, x):
    """(total [B], alpha [B, T + 1, U + 1]) in float64."""
    B, T, U = c["B"], c["T"], c["U"]
    bl, lb = x["blank"].double(), x["label"].double()
    Tb, Ub = x["lens"][:, 0].long(), x["lens"][:, 1].long()
    al = torch.full((B, T + 1, U + 1), NEG, dtype=torch.float64, device=DEV)
    al[:, 0, 0] = 0.0
    bi = torch.arange(B, device=DEV)
    off = torch.arange(U + 1, device=DEV)[None, :] > Ub[:, None]
    if c["form"] != "standard":
        for t in range(1, T + 1):
            stay = al[:, t - 1] + bl[:, t - 1]
            move = al[:, t - 1, :-1] + lb[:, t - 1]
            if c["form"] == "constrained":
                move = move + bl[:, t - 1, 1:]
            al[:, t, 0] = stay[:, 0]
            al[:, t, 1:] = torch.logaddexp(stay[:, 1:], move)
        total = al[bi, Tb, Ub]
    else:
        for d in range(1, T + U):  # the cells with t + u = d
            u = torch.arange(max(0, d - T + 1), min(d, U) + 1, device=DEV)
            t = d - u
            stay = torch.where(t > 0, al[:, (t - 1).clamp(min=0), u] + bl[:, (t - 1).clamp(min=0), u], NEG)
            um = (u - 1).clamp(min=0)
            move = torch.where(u > 0, al[:, t, um] + lb[:, t, um], NEG)
            al[:, t, u] = torch.logaddexp(stay, move)
        total = al[bi, Tb - 1, Ub] + bl[bi, Tb - 1, Ub]
    al.masked_fill_(off[:, None, :], NEG)
    return total, al


def exact(case, seed):
    c, x = case, _inputs(case, seed)
    if c["kind"] == "joiner":
        return dict(logp=_logp64(c, x["w"], x["enc"], x["ctx"].long()))
    if c["kind"] == "transducer":
        total, al = _transducer64(c, x)
        out = dict(total=total, status=None)
        if c["alpha"]:
            out["alpha"] = al[:, :c["T"]] if c["form"] == "standard" else al
        return out
    if c["kind"] == "hyps":
        return dict(tokens=None, num_tokens=None, scores=_hyps64(c, x))
    if c["kind"] == "logadd":
        return dict(tokens=None, num_tokens=None, scores=_logadd64(c, x))
    return dict(tokens=None, num_tokens=None, scores=_search64(c, x), status=None)
