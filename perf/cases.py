"""The work that is timed when this engine is made faster.

A case is one batch of generation calls served to completion through the
public interface: the calls are submitted, the engine is stepped until it is
idle, the tokens are collected. Calls either bring a prompt (``moa_submit``:
prefill, then decode) or a K/V history (``moa_submit_with_history``: decode
only), on one to four resident models. Depth is cut to a few layers of the
real widths so that weights load quickly; one case runs the 1B shape whole.

A few calls of each batch (the "probes") also have their logits captured.
They emit at most two tokens, so that their logits follow from the inputs and
not from a long chain of greedy choices.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2606_03014_amd import Engine, run_feeder

SHAPES = {  # d_model, n_heads, n_kv_heads, head_dim, ffn_dim
    "tiny": (256, 4, 4, 64, 1024),
    "1b": (2048, 32, 8, 64, 8192),
    "8b": (4096, 32, 8, 128, 14336),
}


def _case(name, shape, **kw):
    d, nh, nkv, hd, ffn = SHAPES[shape] if isinstance(shape, str) else shape
    c = dict(name=name, dtype="bf16", layers=2, d=d, heads=nh, kv_heads=nkv, head_dim=hd, ffn=ffn, vocab=4096,
             models=1, skew=0.0,              # calls per model fall off as (m + 1) ** -skew
             flow="step",                     # step | noalloc | one_stream | feeder
             prompts=0, p_lo=1, p_hi=1,       # calls with a prompt, log-uniform lengths
             histories=0, h_lo=1, h_hi=1,     # calls with a K/V history, log-uniform lengths
             pareto=0.0,                      # > 0: history lengths min(h_lo * (1 + Pareto(pareto)), h_hi)
             gen_lo=1, gen_hi=1,              # tokens per call, uniform
             budget=16384, probes=3)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest: a two-layer fp32 mixture of two experts and an aggregator, 48 calls in one pass
        _case("tiny fp32 mixture", "tiny", dtype="f32", flow="feeder", models=3, prompts=16, p_lo=16, p_hi=64,
              gen_lo=8, gen_hi=64, budget=256),
        # one user's short question, every layer of the 1B shape: launches and latency
        _case("1b one question", "1b", layers=16, vocab=32000, prompts=1, p_lo=37, p_hi=37, gen_lo=16, gen_hi=16,
              probes=1),
        # a few calls in a serving loop that may not allocate
        _case("8b four calls noalloc", "8b", flow="noalloc", histories=4, h_lo=300, h_hi=2100, gen_lo=24, gen_hi=32,
              budget=512, probes=1),
        # 512-call expert batch of the 1B shape on four models, popular experts first
        _case("1b four experts decode", "1b", layers=4, models=4, skew=1.2, histories=160, h_lo=64, h_hi=3000,
              gen_lo=8, gen_hi=48, probes=8),
        # the steady state of three 8B experts: 60 to 110 rows per model
        _case("8b three experts decode", "8b", models=3, skew=1.0, histories=250, h_lo=200, h_hi=8000, gen_lo=16,
              gen_hi=40, probes=8),
        # long reasoning stragglers: 512 calls with heavy-tailed histories, the batch draining as they end
        _case("8b stragglers", "8b", histories=512, h_lo=256, h_hi=32768, pareto=1.2, gen_lo=1, gen_hi=40, budget=0,
              probes=8),
        # the tail of such a batch: a handful of very long contexts
        _case("8b long tail", "8b", histories=7, h_lo=12000, h_hi=32001, gen_lo=32, gen_hi=32, budget=0, probes=1),
        # aggregator prompts: the query and every expert's output, in 16k-token chunks
        _case("8b aggregator prefill", "8b", prompts=2, p_lo=9001, p_hi=17003, gen_lo=2, gen_hi=4, probes=2),
        # queries arriving together at three experts: ragged prompts, then decode
        _case("8b prompt burst", "8b", models=3, skew=1.0, prompts=24, p_lo=64, p_hi=3001, gen_lo=8, gen_hi=24,
              probes=8),
        # the same at the 1B shape (head_dim 64)
        _case("1b prompt burst", "1b", layers=4, models=4, skew=1.2, prompts=40, p_lo=32, p_hi=1501, gen_lo=8,
              gen_hi=32, probes=8),
        # the head: a 128k vocabulary behind one layer
        _case("8b head", "8b", layers=1, vocab=128256, histories=96, h_lo=15, h_hi=400, gen_lo=12, gen_hi=12, probes=8),
        # eight query heads per KV head, prompts arriving beside running calls, everything on the caller's stream
        _case("gqa8 mixed one stream", (2048, 16, 2, 128, 5632), layers=3, vocab=8192, models=2, skew=0.5,
              flow="one_stream", prompts=19, p_lo=5, p_hi=777, histories=14, h_lo=33, h_hi=5001, gen_lo=6, gen_hi=30,
              budget=2048, probes=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another batch of the same ranges: widths from 256 to 4096, every grouping of heads, one to four models, 1 to
    512 calls of 1 to 32k positions, prompts, histories or both."""
    while True:
        kind = rng.choice(["prompts", "histories", "histories", "both"])
        if rng.random() < 0.12:
            hd, nkv, gq = 64, rng.choice([1, 2, 4]), rng.choice([1, 2, 4])
            shape = (rng.choice([256, 512]), nkv * gq, nkv, hd, 128 * rng.randint(2, 10))
            dtype, layers = "f32", rng.randint(1, 2)
        else:
            hd = rng.choice([64, 128])
            nkv, gq = rng.choice([(2, 8), (4, 8), (4, 4), (8, 4), (8, 2), (8, 1), (16, 2), (8, 4)])
            shape = (rng.choice([512, 1024, 1536, 2048, 3072, 4096, 4096]), nkv * gq, nkv, hd,
                     _log(rng, 8, 112) * 128)
            dtype, layers = "bf16", rng.randint(1, 3)
        n = _log(rng, 1, 512 if dtype == "bf16" else 40)
        n_p = n if kind == "prompts" else (0 if kind == "histories" else (n + 1) // 2)
        p = sorted(_log(rng, 1, 6000 if dtype == "bf16" else 200) for _ in range(2))
        h = sorted(_log(rng, 1, 32768 if dtype == "bf16" else 500) for _ in range(2))
        g = sorted(_log(rng, 1, 48) for _ in range(2))
        c = _case("", shape, dtype=dtype, layers=layers, vocab=rng.choice([1024, 4096, 8192, 32000]),
                  models=rng.randint(1, 4), skew=round(rng.uniform(0.0, 1.3), 2),
                  flow=rng.choice(["step", "step", "step", "one_stream"]), prompts=n_p, p_lo=p[0], p_hi=p[1],
                  histories=n - n_p, h_lo=h[0], h_hi=h[1], gen_lo=g[0], gen_hi=g[1],
                  budget=rng.choice([512, 2048, 16384]) if n_p else 64)
        del c["name"]
        w, calls = work(c), _calls(c)
        if (w["bytes"] / 3.5e12 + w["flops"] / 4e14 < 0.035 and _kv_tokens(calls) * _kv_row(c) < 5e9
                and c["models"] * _model_elems(c) < 1.4e9 and (dtype == "bf16" or w["flops"] < 3e10)):
            return c


# ------------------------------------------------------------------ the calls of a case

def _calls(c):
    """The case's calls in submission order: dicts of model, kind, n (prompt or history length), gen, probe. Lengths
    are fixed quantiles in a fixed order: only token ids, weights and histories come from the seed."""
    def lengths(n, lo, hi, pareto=0.0):
        q = (np.arange(n) + 0.5) / max(n, 1)
        if pareto:
            v = np.minimum(np.floor(lo * (1.0 - q) ** (-1.0 / pareto)), hi)
        else:
            v = np.rint(np.exp(math.log(lo) + q * (math.log(hi) - math.log(lo))))
        return np.random.default_rng([n, lo, hi]).permutation(v.astype(np.int64))

    n = c["prompts"] + c["histories"]
    rng = np.random.default_rng([n, c["gen_lo"], c["gen_hi"], 7])
    gen = rng.permutation(np.rint(np.linspace(c["gen_lo"], c["gen_hi"], n)).astype(np.int64))
    share = np.arange(1, c["models"] + 1, dtype=np.float64) ** -c["skew"]
    edge = np.rint(np.cumsum(share) / share.sum() * n)
    model = rng.permutation(np.minimum(np.searchsorted(edge, np.arange(n), side="right"), c["models"] - 1))
    kinds = ["prompt"] * c["prompts"] + ["history"] * c["histories"]
    lens = [*lengths(c["prompts"], c["p_lo"], c["p_hi"]), *lengths(c["histories"], c["h_lo"], c["h_hi"], c["pareto"])]
    order = rng.permutation(n)
    calls = [dict(kind=kinds[i], n=int(lens[i]), gen=int(gen[i]), model=int(model[i]), probe=False) for i in order]
    by_len = sorted(range(n), key=lambda i: calls[i]["n"])
    for k in range(min(c["probes"], n)):              # the longest, the shortest and some between
        i = by_len[-1 - k * (n - 1) // max(1, min(c["probes"], n) - 1)] if c["probes"] > 1 else by_len[-1]
        calls[i]["probe"] = True
        if n > 1:
            calls[i]["gen"] = min(calls[i]["gen"], 2)
    return calls


def _kv_tokens(calls):
    return sum(k["n"] + k["gen"] for k in calls)


def _esz(c):
    return 2 if c["dtype"] == "bf16" else 4


def _kv_row(c):
    return c["layers"] * c["kv_heads"] * c["head_dim"] * 2 * _esz(c)


def _layer_elems(c):
    qkv = (c["heads"] + 2 * c["kv_heads"]) * c["head_dim"]
    return 2 * c["d"] + c["d"] * qkv + c["d"] * c["heads"] * c["head_dim"] + 3 * c["d"] * c["ffn"]


def _model_elems(c):
    return 2 * c["vocab"] * c["d"] + c["d"] + c["layers"] * _layer_elems(c)


def _feeder_phases(c):
    """The feeder's batch: every query at every expert, then the aggregator on the query and the answers."""
    calls = _calls(c)
    experts = [dict(k, model=m) for k in calls for m in range(c["models"] - 1)]
    agg = [dict(kind="prompt", n=k["n"] + (c["models"] - 1) * k["gen"], gen=32, model=c["models"] - 1) for k in calls]
    return [experts, agg]


def work(c):
    """Per engine step: the weights of the models that have rows, the K/V that the rows attend to and append, the
    logits; every prompt position and decoded token through the matrices and the causal attention."""
    nh, hd, e = c["heads"], c["head_dim"], _esz(c)
    byts = flops = 0.0
    for calls in (_feeder_phases(c) if c["flow"] == "feeder" else [_calls(c)]):
        left = [k["n"] if k["kind"] == "prompt" else 0 for k in calls]
        gen = [0] * len(calls)
        while any(g < k["gen"] for g, k in zip(gen, calls)):
            budget, models = c["budget"], set()
            for i, k in enumerate(calls):
                if gen[i] >= k["gen"]:
                    continue
                if left[i] > 0:
                    if budget <= 0:
                        continue
                    rows = min(left[i], budget)
                    pos = k["n"] - left[i]
                    left[i] -= rows
                    budget -= rows
                    emits = left[i] == 0
                else:
                    rows, emits, pos = 1, True, k["n"] + gen[i] - (k["kind"] == "prompt")
                models.add(k["model"])
                byts += (pos + 2 * rows) * _kv_row(c) + rows * c["d"] * e
                flops += rows * 2.0 * c["layers"] * _layer_elems(c)
                flops += 4.0 * nh * hd * c["layers"] * (rows * pos + rows * (rows + 1) / 2)
                if emits:
                    gen[i] += 1
                    byts += 4.0 * c["vocab"]
                    flops += 2.0 * c["vocab"] * c["d"]
            byts += len(models) * (c["layers"] * _layer_elems(c) + c["vocab"] * c["d"]) * e
    return {"bytes": byts, "flops": flops}


# ------------------------------------------------------------------ inputs

def _weights(c, seed, m):
    """One model's packed tensors (embed, layers, final norm, LM head) on the GPU: N(0, 0.02^2), unit gains."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 16 + m)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    w = torch.empty(_model_elems(c), dtype=dt, device="cuda")
    for part in w.split(1 << 26):
        part.copy_(torch.empty(part.numel(), device="cuda").normal_(0.0, 0.02, generator=g))
    d, at = c["d"], c["vocab"] * c["d"]
    qo = c["d"] * (c["heads"] + 2 * c["kv_heads"]) * c["head_dim"] + c["d"] * c["heads"] * c["head_dim"]
    for _ in range(c["layers"]):
        w[at:at + d] = 1
        w[at + d + qo:at + 2 * d + qo] = 1
        at += _layer_elems(c)
    w[at:at + d] = 1
    return w


def prepare(c, seed):
    calls = _calls(c)
    shape = SimpleNamespace(n_layers=c["layers"], d_model=c["d"], n_heads=c["heads"], n_kv_heads=c["kv_heads"],
                            head_dim=c["head_dim"], ffn_dim=c["ffn"], vocab=c["vocab"], rope_theta=10000.0,
                            rms_eps=1e-5)
    every = [k for ph in _feeder_phases(c) for k in ph] if c["flow"] == "feeder" else calls
    longest = max(k["n"] + k["gen"] for k in every)
    consts = SimpleNamespace(kv_block_size=16, num_kv_blocks=sum((k["n"] + k["gen"]) // 16 + 1 for k in every),
                             max_num_seqs=max(len(calls), 16 if c["flow"] == "feeder" else 1),
                             max_prefill_tokens=c["budget"], max_model_len=max(longest, 2))
    eng = Engine(shape, c["dtype"], consts, c["models"], one_stream=c["flow"] == "one_stream",
                 token_store=1 << 20, block_store=1 << 18)
    for m in range(c["models"]):
        eng.load(_weights(c, seed, m).view(torch.uint8).cpu().numpy())
    rng = np.random.default_rng([int(seed), 5])
    for k in calls:
        k["tokens"] = rng.integers(0, c["vocab"], k["n"] if k["kind"] == "prompt" else 1).astype(np.int32)
        k["logits"] = torch.zeros(k["gen"], c["vocab"], pin_memory=True) if k["probe"] else None
    return {"case": c, "eng": eng, "calls": calls}


def run(s):
    c, eng, calls = s["case"], s["eng"], s["calls"]
    if c["flow"] == "feeder":
        return _run_feeder(c, eng, calls)
    ids = []
    for k in calls:
        if k["kind"] == "prompt":
            ids.append(eng.submit(k["tokens"], k["model"], k["gen"]))
        else:
            ids.append(eng.submit_with_history(k["model"], int(k["tokens"][0]), k["n"], k["gen"]))
        if k["probe"]:
            eng.capture_logits(ids[-1], k["logits"].view(-1).numpy())
    step = eng.step_noalloc if c["flow"] == "noalloc" else eng.step
    while step().step >= 0:
        pass
    got = {r[0]: r[3] for r in eng.collect()}
    eng.sync()                                        # the captured logits are in host memory
    probes = [k["logits"] for k in calls if k["probe"]]
    return {"tokens": np.concatenate([got[i] for i in ids]), "first": [x[0] for x in probes],
            "later": [x[1:] for x in probes if len(x) > 1]}


def _run_feeder(c, eng, calls):
    n_e = c["models"] - 1
    wl = SimpleNamespace(prompts=[k["tokens"] for k in calls], experts=[tuple(range(n_e))] * len(calls),
                         n_queries=len(calls), n_experts=n_e, agg_max_new=32,
                         expert_requests=lambda: [(q, e, k["gen"]) for q, k in enumerate(calls) for e in range(n_e)])

    def on_submit(rid, q, model, gen):
        if calls[q]["probe"] and model == 0:
            eng.capture_logits(rid, calls[q]["logits"].view(-1).numpy())

    res = run_feeder(eng, wl, list(range(n_e)), agg_model=n_e, on_submit=on_submit)
    eng.sync()
    probes = [k["logits"] for k in calls if k["probe"]]
    return {"tokens": np.concatenate([res.outputs[(q, m)] for q in range(len(calls)) for m in range(n_e + 1)]),
            "first": [x[0] for x in probes], "later": [x[1:] for x in probes if len(x) > 1]}


def tolerance(c):
    # Four times the error of the probes' logits (2-norm) against the same path in 64 bits, measured over the listed
    # cases: at most 8e-7 in fp32 and 9.4e-4 in bf16 (16 layers; 5.5e-4 over two to four). The bf16 K/V cache is rounded
    # on both sides; what is left is fp32 sums, and the few K/V elements whose rounding to bf16 falls the other way.
    # Tokens may differ where the two largest logits are closer than that.
    if c["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-5, "differ": 0.01}
    return {"rel": 4e-3, "max": 4e-2, "differ": 0.01}


# ------------------------------------------------------------------ the same in 64 bits

def _mix(x):
    for shift, mul in ((16, 0x7FEB352D), (15, 0x846CA68B)):
        x = ((x ^ (x >> shift)) * mul) & 0xFFFFFFFF
    return x ^ (x >> 16)


def _history(c, rid, layer, kv, n):
    """The device-filled history [n, kv_heads, head_dim]: values in [-1, 1) from a hash of request, layer, K or V,
    position and element."""
    p = torch.arange(n, device="cuda").view(-1, 1)
    r = torch.arange(c["kv_heads"] * c["head_dim"], device="cuda").view(1, -1)
    u = _mix(((rid * 0x9E3779B9) & 0xFFFFFFFF) ^ _mix(((layer * 2 + kv) << 24) ^ p) ^ ((r * 0x85EBCA6B) & 0xFFFFFFFF))
    v = (u >> 8).double() / 8388608.0 - 1.0
    return _store(c, v).view(n, c["kv_heads"], c["head_dim"])


def _store(c, v):
    return v.to(torch.bfloat16 if c["dtype"] == "bf16" else torch.float32).double()


def _forward(c, w, call, rid):
    """Logits of the call's first emitted token."""
    d, nh, nkv, hd, ffn, V = c["d"], c["heads"], c["kv_heads"], c["head_dim"], c["ffn"], c["vocab"]
    hist = call["n"] if call["kind"] == "history" else 0
    tok = torch.from_numpy(call["tokens"]).long().cuda()
    T, at = len(tok), V * d

    def take(*shape):
        nonlocal at
        n = math.prod(shape)
        at += n
        return w[at - n:at].double().view(*shape)

    def norm(x, g):
        return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + 1e-5) * g

    def rope(x):
        ang = (hist + torch.arange(T, device="cuda").double()).view(-1, 1, 1) \
            * 10000.0 ** (-2.0 * torch.arange(hd // 2, device="cuda").double() / hd)
        a, b = x[..., :hd // 2], x[..., hd // 2:]
        return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)

    x = w[:at].view(V, d)[tok].double()
    for layer in range(c["layers"]):
        y = norm(x, take(d))
        q = rope((y @ take(nh * hd, d).t()).view(T, nh, hd))
        k = _store(c, rope((y @ take(nkv * hd, d).t()).view(T, nkv, hd)))
        v = _store(c, (y @ take(nkv * hd, d).t()).view(T, nkv, hd))
        if hist:
            k = torch.cat([_history(c, rid, layer, 0, hist), k])
            v = torch.cat([_history(c, rid, layer, 1, hist), v])
        o = torch.empty(T, nh, hd, dtype=torch.float64, device="cuda")
        key = torch.arange(len(k), device="cuda")
        for h in range(nh):
            kh, vh = k[:, h * nkv // nh].contiguous(), v[:, h * nkv // nh].contiguous()
            for r0 in range(0, T, 4096):
                s = q[r0:r0 + 4096, h] @ kh.t() / math.sqrt(hd)
                s.masked_fill_(key > hist + r0 + torch.arange(len(s), device="cuda").view(-1, 1), -math.inf)
                o[r0:r0 + 4096, h] = torch.softmax(s, -1) @ vh
        x = x + o.view(T, nh * hd) @ take(d, nh * hd).t()
        y = norm(x, take(d))
        gate = y @ take(ffn, d).t()
        up = y @ take(ffn, d).t()
        x = x + (torch.nn.functional.silu(gate) * up) @ take(d, ffn).t()
    y = norm(x[-1:], take(d))
    return (y @ take(V, d).t())[0]


def exact(c, seed):
    """First-token logits of the probes. What follows hangs on greedy choices and has no value of its own."""
    calls = _calls(c)
    rng = np.random.default_rng([int(seed), 5])
    for k in calls:
        k["tokens"] = rng.integers(0, c["vocab"], k["n"] if k["kind"] == "prompt" else 1).astype(np.int32)
    first = {}
    for m in range(c["models"]):
        w = None
        for rid, k in enumerate(calls):
            if k["probe"] and m == (0 if c["flow"] == "feeder" else k["model"]):
                w = _weights(c, seed, m) if w is None else w
                first[rid] = _forward(c, w, k, rid)
    return {"tokens": None, "first": [first[i] for i in sorted(first)], "later": None}
