"""Performance cases of the inference-time hot path: what is timed, on which sizes, and how far two
correct results may lie apart.

Every case is one piece of work that a serving program hands to the library through its public
binding, on a slice of a model's layers (the layers of a model are alike; a slice of a few keeps a
state small while its working set still exceeds the last-level cache together with the states
that a measurement takes in turn):

  chunk    a document chunk is materialized: per layer the K/V projection with rotary embedding and
           the chunk's own causal attention; optionally the finished blob is compressed for the store
  prefill  a batch of questions arrives over chunks that are resident: cache assembly, per layer the
           question's K/V projection and its attention over chunks and question
  decode   tokens are generated: cache assembly, then one recorded graph per step (tail advance, per
           layer the new token's K/V projection and its attention over everything)
  stream   two instances one after the other: the chunks of the next are loaded from pinned host
           memory beside the current one's question and decode steps
  request  one whole small request without graphs: load, assembly, question, decode steps

Model shapes and workload sizes are those of the repository's benchmark and tests (the 3B, 8B and 70B
layer shapes, chunks of about a thousand tokens, short questions, a pool of chunks shared by a batch).
"""
from __future__ import annotations

import math
import random

import torch

from paper_2512_22195_amd import binding as mk

# query heads, KV heads, head_dim, hidden, element type, rotary base
MODELS = {
    "tiny": (4, 2, 64, 256, "f32", 10000.0),
    "3b": (24, 8, 128, 3072, "bf16", 500000.0),
    "8b": (32, 8, 128, 4096, "bf16", 500000.0),
    "70b": (64, 8, 128, 8192, "bf16", 500000.0),
}


def _case(name, kind, model, layers, *, batch=1, chunks=1, tokens=(1000, 1000), pool=0, fmt="plain", question=(64, 64), steps=0,
          compress=False):
    return {"name": name, "kind": kind, "model": model, "layers": layers, "batch": batch, "chunks": chunks,
            "tok_min": tokens[0], "tok_max": tokens[1], "pool": pool, "fmt": fmt, "q_min": question[0], "q_max": question[1],
            "steps": steps, "compress": compress}


def listed():
    return [
        # The smallest request there is: one fp32 layer of the tiny configuration, two chunks of 256
        # tokens, a 32-token question, eight tokens.  All launches, copies and host calls.
        _case("request_tiny_f32", "request", "tiny", 1, chunks=2, tokens=(256, 256), question=(32, 32), steps=8),
        # Short contexts: three users of a 3B model, a few short passages each, ragged.  Latency.
        _case("decode_3b_b3_short", "decode", "3b", 8, batch=3, chunks=3, tokens=(90, 310), question=(9, 33), steps=16),
        # The store is filled: one chunk of ordinary length, kept in compressed form.
        _case("chunk_8b_compressed", "chunk", "8b", 8, tokens=(1000, 1000), compress=True),
        # The same for the large model, kept as it is.
        _case("chunk_70b", "chunk", "70b", 4, tokens=(1000, 1000)),
        # A long document section of odd length.
        _case("chunk_8b_long", "chunk", "8b", 4, tokens=(3501, 3501)),
        # One user, ten retrieved chunks, a 64-token question: the time to the first token.
        _case("prefill_8b_b1", "prefill", "8b", 8, chunks=10, question=(64, 64)),
        # Sixteen users with questions of 32 to 128 tokens, five chunks each out of a pool of 200.
        _case("prefill_8b_b16_pool", "prefill", "8b", 4, batch=16, chunks=5, pool=200, question=(32, 128)),
        # Four users of the large model over 20 000 tokens each.
        _case("prefill_70b_b4", "prefill", "70b", 4, batch=4, chunks=20, question=(128, 128)),
        # The same three loads while tokens are generated.
        _case("decode_8b_b1", "decode", "8b", 8, chunks=10, question=(64, 64), steps=8),
        _case("decode_8b_b16_pool", "decode", "8b", 4, batch=16, chunks=5, pool=200, question=(32, 128), steps=8),
        _case("decode_70b_b4", "decode", "70b", 4, batch=4, chunks=20, question=(128, 128), steps=8),
        # Chunks in compressed form come from host memory, the next instance's beside the current one.
        _case("stream_8b_e4m3", "stream", "8b", 4, chunks=10, fmt="e4m3", question=(64, 64), steps=32),
    ]


# ---------------------------------------------------------------- what a case consists of

def _dims(case):
    Hq, Hkv, D, Hd, dtype, base = MODELS[case["model"]]
    return Hq, Hkv, D, Hd, dtype, base, 4 if dtype == "f32" else 2


def _batch(case):
    """Chunk lengths (by chunk id), chunk ids of every instance, question lengths; fixed by the case's sizes."""
    r = random.Random(repr([case[k] for k in ("model", "batch", "chunks", "tok_min", "tok_max", "pool", "q_min", "q_max")]))
    B, n = case["batch"], case["chunks"]
    ids = [r.sample(range(case["pool"]), n) if case["pool"] else list(range(b * n, b * n + n)) for b in range(B)]
    lens = {c: r.randint(case["tok_min"], case["tok_max"]) for c in sorted({c for i in ids for c in i})}
    return lens, ids, [r.randint(case["q_min"], case["q_max"]) for _ in range(B)]


def work(case):
    Hq, Hkv, D, Hd, _, _, s = _dims(case)
    lens, ids, qs = _batch(case)
    NL, B, S = case["layers"], case["batch"], case["steps"]
    weights = 2 * Hkv * D * Hd * s
    row = 2 * Hkv * D                                     # K and V elements of one token

    def proj(rows):                                       # hidden rows in, K/V rows out
        return rows * (Hd + row) * s, 2.0 * rows * Hd * row

    def pages(distinct=True):                             # bytes of the chunk pages one layer reads
        toks = sum(lens.values()) if distinct else sum(lens[c] for i in ids for c in i)
        return toks * row * (1 if case["fmt"] == "e4m3" else s)

    def question():
        b, f = proj(sum(qs))
        keys = sum(q * sum(lens[c] for c in i) + q * (q + 1) / 2 for q, i in zip(qs, ids))
        return b + weights + pages() + 2 * sum(qs) * Hq * D * s, f + 4.0 * D * Hq * keys

    def steps():
        b, f = proj(B)
        keys = sum(sum(lens[c] for c in i) + q for q, i in zip(qs, ids)) * S + B * S * (S + 1) / 2
        tail = (sum(qs) * S + B * S * (S - 1) / 2) * row * s
        return S * (b + weights + pages() + 2 * B * Hq * D * s) + tail, S * f + 4.0 * D * Hq * keys

    if case["kind"] == "chunk":
        T = case["tok_max"]
        b, f = proj(T)
        b += weights + 2 * T * Hq * D * s + (T * row if case["compress"] else 0)
        f += 4.0 * D * Hq * T * (T + 1) / 2
    elif case["kind"] == "prefill":
        b, f = question()
    elif case["kind"] == "decode":
        b, f = steps()
    else:                                                 # whole instances, the loaded bytes once more
        (b0, f0), (b1, f1) = question(), steps()
        n = 2 if case["kind"] == "stream" else 1
        b, f = n * (b0 + b1 + pages(False)), n * (f0 + f1)
    return {"bytes": NL * b, "flops": NL * f}


def _cost(case):
    w = work(case)
    return max(w["bytes"] / 6e12, w["flops"] / 1e15)


def tolerance(case):
    """Four times the distance from a float64 computation on the same inputs: fp32 1.8e-7 of the norm and
    8e-7 of a value; bf16 2.3e-3 of the norm (K, V and outputs are stored in bf16, the weights of the sums are
    rounded to it), 1e-2 of a value over whole caches and 3.3e-2 in a chunk's first rows, which see few keys."""
    if case["model"] == "tiny":
        return {"rel": 1e-6, "max": 4e-6}
    if case["kind"] != "chunk":
        return {"rel": 1e-2, "max": 4e-2}
    if case["compress"]:                                  # a stored value rounded the other way may take another code
        return {"rel": 1e-2, "max": 0.13, "differ": 2e-4}
    return {"rel": 1e-2, "max": 0.13}


# ---------------------------------------------------------------- drawn cases

def draw(rng):
    most = max(_cost(c) for c in listed())

    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def span(lo, hi):                                     # half of the draws uniform, half ragged
        a = log(lo, hi)
        return (a, a) if rng.random() < 0.5 else (max(lo, int(a * rng.uniform(0.3, 1.0))), a)

    while True:
        kind = rng.choice(["chunk", "chunk", "prefill", "prefill", "decode", "decode", "decode", "stream", "request"])
        model = "tiny" if kind == "request" else rng.choice(["3b", "8b", "8b", "70b"])
        layers = 1 if kind == "request" else 4
        if kind == "chunk":
            T = log(64, 4096)
            case = _case("", kind, model, layers, tokens=(T, T), compress=rng.random() < 0.4)
        elif kind == "request":
            case = _case("", kind, model, layers, chunks=rng.randint(1, 4), tokens=span(40, 600), question=span(4, 60), steps=rng.randint(2, 12))
        elif kind == "stream":
            case = _case("", kind, model, layers, chunks=rng.randint(2, 10), tokens=span(200, 1200), fmt=rng.choice(["plain", "e4m3"]),
                         question=span(8, 128), steps=rng.randint(8, 32))
        else:
            batch = log(1, 24)
            chunks = rng.randint(1, 20)
            case = _case("", kind, model, layers, batch=batch, chunks=chunks, tokens=span(64, 1500),
                         pool=rng.choice([0, 0, 40, 200]) if batch > 1 else 0, fmt=rng.choice(["plain", "plain", "e4m3"]),
                         question=span(4, 200), steps=rng.choice([4, 8, 12]) if kind == "decode" else 0)
        lens, _, _ = _batch(case)
        held = case["layers"] * sum(lens.values()) * 4 * MODELS[model][1] * MODELS[model][2]
        if _cost(case) <= most and held <= 12e9:
            del case["name"]
            return case


# ---------------------------------------------------------------- state and pass

_STREAMS = None


def _streams():
    """One compute and one load stream for every context of the process, as the library advises."""
    global _STREAMS
    if _STREAMS is None:
        _STREAMS = (torch.cuda.Stream(), torch.cuda.Stream())
    return _STREAMS


class _State:
    pass


def prepare(case, seed):
    Hq, Hkv, D, Hd, dtype, base, _ = _dims(case)
    lens, ids, qs = _batch(case)
    NL, B, S, kind = case["layers"], case["batch"], case["steps"], case["kind"]
    st = _State()
    st.case, st.kind, st.layers, st.steps, st.q_lens = case, kind, NL, S, qs
    dev, tdt = torch.device("cuda:0"), torch.float32 if dtype == "f32" else torch.bfloat16
    max_tail = (max(qs) + S + 7) // 8 * 8 if kind != "chunk" else 64
    cfg = mk.make_config(NL, Hq, Hkv, D, Hd, dtype, base, max_batch=B, max_pages=case["chunks"], max_tail_tokens=max_tail)
    st.ctx = ctx = mk.Context(cfg, *_streams(), device=dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))

    def normal(*shape, scale=1.0):
        return torch.empty(shape, dtype=tdt, device=dev).normal_(0.0, scale, generator=gen)

    with torch.cuda.stream(ctx.compute_stream):
        st.w = normal(NL, 2, Hkv * D, Hd, scale=Hd ** -0.5)
        if kind == "chunk":
            st.T = T = case["tok_max"]
            st.x, st.q = normal(NL, T, Hd), normal(NL, T, Hq, D)
            st.blob = torch.empty((NL, 2, Hkv, T, D), dtype=tdt, device=dev)
            st.out = torch.empty_like(st.q)
            st.packed = torch.empty(mk.compressed_blob_bytes(cfg, T), dtype=torch.uint8, device=dev) if case["compress"] else None
            return st
        fmt = mk.PAGE_E4M3 if case["fmt"] == "e4m3" else mk.PAGE_PLAIN

        def blob(n):                                      # a chunk as the store holds it
            v = normal(NL, 2, Hkv, n, D)
            if fmt == mk.PAGE_PLAIN:
                return v.view(torch.uint8).view(-1)
            packed = torch.empty(mk.compressed_blob_bytes(cfg, n), dtype=torch.uint8, device=dev)
            ctx.compress(v, n, packed)
            return packed

        n_inst = 2 if kind == "stream" else 1             # instance batches one pass serves, one after the other
        st.table = ctx.new_table()
        st.tails = [ctx.new_tail() for _ in range(n_inst)]
        st.host, st.slots, st.pages = [], [], []
        for _ in range(n_inst):
            slots = {c: blob(n) for c, n in lens.items()}
            if kind in ("stream", "request"):
                st.host.append({c: torch.empty(v.shape, dtype=torch.uint8, pin_memory=True).copy_(v) for c, v in slots.items()})
                for v in slots.values():
                    v.zero_()
            st.slots.append(slots)
            st.pages.append([[(slots[c], lens[c], fmt) for c in i] for i in ids])
        st.lens = lens
        nq = sum(qs)
        if kind != "decode":
            st.x_q, st.q_q = normal(n_inst, NL, nq, Hd), normal(n_inst, NL, nq, Hq, D)
            st.o_q = torch.empty_like(st.q_q)
        if kind != "prefill":
            st.x_d, st.q_d = normal(n_inst, S, NL, B, Hd), normal(n_inst, S, NL, B, Hq, D)
            st.o_d = torch.empty_like(st.q_d)
        if kind == "decode":                              # the questions' rows, as a prefill left them
            st.tails[0].normal_(0.0, 1.0, generator=gen)
        if kind in ("decode", "stream"):
            ctx.assemble(st.pages[0], qs, st.table)
            st.graphs = [[_record(st, i, k) for k in range(S)] for i in range(n_inst)]
    return st


def _record(st, i, k):
    st.ctx.graph_begin()
    _step(st, i, k)
    return st.ctx.graph_end()


def _step(st, i, k):
    """Decode step k of instance batch i: one more tail row, every layer."""
    ctx, tail = st.ctx, st.tails[i]
    ctx.advance(st.table, 1)
    for l in range(st.layers):
        ctx.decode_step(l, st.x_d[i, k, l], st.w[l, 0], st.w[l, 1], st.q_d[i, k, l], st.table, tail[l, 0], tail[l, 1], st.o_d[i, k, l])


def _question(st, i):
    ctx, tail = st.ctx, st.tails[i]
    for l in range(st.layers):
        ctx.materialize_tail(st.x_q[i, l], st.w[l, 0], st.w[l, 1], st.table, -1, tail[l, 0], tail[l, 1])
        ctx.prefill_attn(l, st.q_q[i, l], st.table, tail[l, 0], tail[l, 1], st.o_q[i, l])


def _load(st, i):
    return [st.ctx.load(st.host[i][c], n, st.slots[i][c]) for c, n in st.lens.items()]


def run(st):
    ctx = st.ctx
    if st.kind == "chunk":
        for l in range(st.layers):
            ctx.materialize(st.x[l], st.w[l, 0], st.w[l, 1], st.T, 0, st.blob[l, 0], st.blob[l, 1], st.T)
            ctx.chunk_attn(l, st.q[l], st.blob, st.T, st.out[l])
        if st.packed is None:
            return {"blob": st.blob, "out": st.out}
        ctx.compress(st.blob, st.T, st.packed)
        return {"blob": st.blob, "out": st.out, "packed": st.packed}
    if st.kind == "prefill":
        ctx.assemble(st.pages[0], st.q_lens, st.table)
        _question(st, 0)
        return {"out": st.o_q, "tail": st.tails[0]}
    if st.kind == "decode":
        ctx.assemble(st.pages[0], st.q_lens, st.table)
        for g in st.graphs[0]:
            ctx.graph_launch(g)
        return {"out": st.o_d, "tail": st.tails[0]}
    tickets = _load(st, 0)
    for i in range(len(st.pages)):
        for t in tickets:
            ctx.wait(t)
        ctx.assemble(st.pages[i], st.q_lens, st.table)
        if i + 1 < len(st.pages):
            tickets = _load(st, i + 1)
        _question(st, i)
        for k in range(st.steps):
            if st.kind == "stream":
                ctx.graph_launch(st.graphs[i][k])
            else:
                _step(st, i, k)
    return {"out_q": st.o_q, "out_d": st.o_d, "tails": st.tails}
