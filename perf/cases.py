"""The work that users of this library have it do, as timed cases: whole sentences, batches and images decoded through the
public entry points, an encoder pass alone, a serving loop of single steps, and the scores of a forced target.

Weights are random of the shapes of the library's workloads (N(0, 0.02), LayerNorm gains about 1), drawn on the GPU.  Random
weights are never sure of a token, so the target-side position table carries, at twice the strength of the token
embeddings, the embedding of the token to be said there: the scores then have a clear first, as a trained model's have, and
tokens do not depend on the rounding of a sum.  The tokens to be said come in runs (text) or as a slow walk through the
intensities (images), so that exact and approximate verification accept blocks of the lengths that the paper reports.
Lengths and schedules depend on the case alone: every seed is the same amount of work on other weights, sources and tokens.
"""
import math

import numpy as np
import torch

from paper_1811_03115_amd import binding

MODELS = {
    "tiny": dict(layers=2, d=64, heads=4, ff=256, vocab=256, k=4, dtype="f32", eos=2),
    "base": dict(layers=6, d=512, heads=8, ff=2048, vocab=32000, k=8, dtype="bf16", eos=2),
    "big": dict(layers=6, d=1024, heads=16, ff=4096, vocab=32768, k=10, dtype="bf16", eos=2),
    "image": dict(layers=6, d=512, heads=8, ff=2048, vocab=256, k=10, dtype="bf16", eos=-1),
}
# call: what run() does with a state; batch sequences, the longest source, the largest output budget, the block size k;
# mean: the mean accepted block (imposed: by a schedule, otherwise the mean run length of the tokens to be said);
# two_phase, top_n, eps: bpd_set_two_phase, bpd_set_top_n, bpd_set_acceptance; local: bpd_set_local_attention (query block and memory)
DEFAULTS = dict(call="decode", model="big", batch=1, source=27, target=128, k=10, mean=5, imposed=True, two_phase=False, top_n=1, eps=0, local=0)


def case(**kw):
    return dict(DEFAULTS, **kw)


def listed():
    return [
        # a small fp32 model decoding one short sentence: a chain of launches and nothing else
        case(name="tiny-sentence", model="tiny", source=16, target=32, k=4, mean=3, imposed=False),
        # one sentence with the base and the big model, k and accepted lengths as in the paper's best runs
        case(name="base-sentence", model="base", source=32, target=64, k=8, mean=4),
        case(name="big-sentence", source=27, target=128, k=10, mean=5),
        # greedy decoding, which the paper's speedups are quoted against
        case(name="big-greedy", source=27, target=33, k=1, mean=1),
        # a serving loop that calls step by step for a few requests at once, exact verification
        case(name="big-serving-steps", call="steps", batch=5, source=50, target=60, k=8, mean=4, imposed=False),
        # offline translation: ragged batches; the full table and the two-phase variant
        case(name="big-batch32", batch=32, source=128, target=128, k=10, mean=3),
        case(name="big-batch32-two-phase", batch=32, source=128, target=128, k=10, mean=3, two_phase=True),
        # an odd batch of the base model with top-2 selection
        case(name="base-batch13-top2", model="base", batch=13, source=60, target=70, k=6, mean=6, imposed=False, top_n=2),
        # the encoder and the first invocation alone, and the scores that follow: what a request pays before its first step
        case(name="big-encode32", call="encode", batch=32, source=128, target=128, k=10),
        # super-resolution: 3072 intensities per image with approximate verification, full and 1D local self-attention
        case(name="image-batch8", model="image", batch=8, source=192, target=3072, k=10, mean=7, imposed=False, eps=2),
        case(name="image-local", model="image", batch=3, source=192, target=3072, k=8, mean=7, imposed=False, eps=2, local=256),
        # a given target forced through the model in blocks, and the scores of its last block for every head
        case(name="base-scores", call="scores", model="base", batch=4, source=40, target=48, k=8),
    ]


def draw(rng):
    def log(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    while True:
        kind = rng.choice(["text", "text", "text", "steps", "encode", "image", "scores"])
        if kind == "image":
            c = case(model="image", batch=log(1, 8), source=192, target=log(64, 3072), k=rng.randint(2, 10), mean=7, imposed=rng.random() < 0.3, eps=2,
                     local=rng.choice([0, 0, 128, 256]))
        else:
            model = rng.choice(["tiny", "base", "base", "big", "big", "big"])
            most = 8 if model == "tiny" else 64
            k = rng.randint(1, MODELS[model]["k"])
            c = case(call={"text": "decode"}.get(kind, kind), model=model, batch=log(1, most), source=log(4, 128), target=log(8, 128), k=k, mean=rng.randint(1, k),
                     imposed=rng.random() < 0.6)
            if kind == "scores":
                c.update(model="base" if model == "big" else model, batch=log(1, 6), k=min(k, MODELS["base"]["k"] if model != "tiny" else 4))
            elif kind == "text" and not c["imposed"] and rng.random() < 0.25:
                c["top_n"] = rng.randint(2, 3)
            if kind in ("text", "steps"):
                c["two_phase"] = rng.random() < 0.25
        c["mean"] = min(c["mean"], c["k"])
        w, most = work(c), [work(x) for x in listed()]
        if w["bytes"] <= max(x["bytes"] for x in most) and w["flops"] <= max(x["flops"] for x in most):
            return c


def _lengths(c):
    """Source lengths and output budgets: one sentence or images as given; batches of text ragged (log-normal, median 27)."""
    b, s, t = c["batch"], c["source"], c["target"]
    if b == 1 or c["model"] == "image" or c["call"] in ("encode", "scores"):
        return np.full(b, s, np.int32), np.full(b, t, np.int32)
    rng = np.random.default_rng(b * 1000 + s)
    n = np.clip(np.rint(np.exp(rng.normal(math.log(27), 0.6, b))), 1, s).astype(np.int32)
    return n, np.clip(np.rint(1.1 * n) + 4, 1, t).astype(np.int32)


def _schedule(c, rows):
    """Accepted lengths [rows, batch] in 1..k: truncated geometric with about the asked mean."""
    k, mean = c["k"], c["mean"]
    if mean <= 1 or mean >= k:
        return np.full((rows, c["batch"]), max(1, min(k, mean)), np.int32)
    a, lo, hi = np.arange(1, k + 1), 1e-6, 1e6
    for _ in range(100):
        r = math.sqrt(lo * hi)
        p = r ** (a - 1.0) / np.sum(r ** (a - 1.0))
        lo, hi = (r, hi) if float(p @ a) < mean else (lo, r)
    return np.random.default_rng(k * 100 + mean).choice(a, size=(rows, c["batch"]), p=p).astype(np.int32)


def _text(c, n, gen):
    """The n tokens to be said, one per target position, as an int64 tensor on the GPU."""
    m = MODELS[c["model"]]
    rng = np.random.default_rng(n + 7)
    if c["model"] == "image":                      # intensities: steps of -1 .. 1, reflected at both ends
        start = int(torch.randint(0, 256, (1,), device="cuda", generator=gen))
        v = (start + np.cumsum(rng.integers(-1, 2, n))) % 510
        return torch.from_numpy(np.where(v > 255, 510 - v, v)).cuda()
    runs = np.repeat(np.arange(n), rng.geometric(1.0 / c["mean"], n))[:n]
    said = torch.randint(3, m["vocab"], (n,), device="cuda", generator=gen)
    return said[torch.from_numpy(runs).cuda()]


def _weights(c, m, slots, gen):
    dtype = torch.bfloat16 if m["dtype"] == "bf16" else torch.float32
    d, f, v, k = m["d"], m["ff"], m["vocab"], m["k"]
    w = {}

    def add(name, *shape, mean=0.0):
        w[name] = torch.randn(shape, device="cuda", generator=gen).mul_(0.02).add_(mean).to(dtype)

    def ln(p):
        add(p + ".g", d, mean=1.0)
        add(p + ".b", d)

    def ffn(p):
        add(p + ".w1", d, f), add(p + ".b1", f), add(p + ".w2", f, d), add(p + ".b2", d)

    add("emb", v, d)
    add("pos_src", c["source"], d)
    for side in ("enc", "dec"):
        for i in range(m["layers"]):
            p = f"{side}.{i}"
            ln(p + ".ln1"), ln(p + ".ln2")
            if side == "dec":
                ln(p + ".ln3")
            for a in ("self", "cross") if side == "dec" else ("self",):
                for x in ("wq", "wk", "wv", "wo"):
                    add(f"{p}.{a}.{x}", d, d)
            ffn(p + ".ffn")
        ln(side + ".lnf")
    add("head.w1", k, d, f), add("head.b1", k, f), add("head.w2", k, f, d), add("head.b2", k, d)
    w["pos_tgt"] = (w["emb"][_text(c, slots, gen)].float() * (2 * math.sqrt(d))).to(dtype)
    return w


def prepare(case, seed):
    c = case
    m = MODELS[c["model"]]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    n, budget = _lengths(c)
    s = int(n.max())
    ctx = binding.Context(binding.make_config(
        n_enc_layers=m["layers"], n_dec_layers=m["layers"], d_model=m["d"], n_heads=m["heads"], d_ff=m["ff"], vocab=m["vocab"], k_max=m["k"],
        max_batch=c["batch"], max_src_len=c["source"], max_out_len=c["target"], dtype=binding.BPD_F32 if m["dtype"] == "f32" else binding.BPD_BF16,
        eos_id=m["eos"], pad_id=0, ln_eps=1e-6))
    ctx.bpd_load_weights(_weights(c, m, c["target"] + m["k"] + 1, gen))
    if c["two_phase"]:
        ctx.bpd_set_two_phase(True)
    if c["top_n"] > 1:
        ctx.bpd_set_top_n(c["top_n"])
    if c["eps"]:
        ctx.bpd_set_acceptance(c["eps"], 1)
    if c["local"]:
        ctx.bpd_set_local_attention(c["local"], c["local"])
    rng = np.random.default_rng(int(seed))
    if c["model"] == "image":
        src = rng.integers(0, m["vocab"], (c["batch"], s)).astype(np.int32)
    else:                                          # word frequencies: rank^-1.1
        rank = np.arange(1, m["vocab"] - 2) ** -1.1
        cdf = np.cumsum(rank / rank.sum())
        src = (3 + np.minimum(np.searchsorted(cdf, rng.random((c["batch"], s))), m["vocab"] - 4)).astype(np.int32)
        src[np.arange(s)[None, :] >= n[:, None]] = 0
    state = dict(c=c, ctx=ctx, src=src, n=n, budget=budget)
    if c["call"] == "decode" and c["imposed"]:
        state["schedule"] = _schedule(c, int(budget.max()))
    elif c["call"] == "steps":
        steps = _steps(c)
        state["accepted"] = torch.zeros((steps, c["batch"]), dtype=torch.int32, device="cuda")
        state["imposed"] = torch.from_numpy(_schedule(c, steps)).cuda() if c["imposed"] else [None] * steps
    elif c["call"] == "scores":                    # the target in blocks of k, proposed one after the other
        blocks = max(1, c["target"] // c["k"])
        forced = rng.integers(3, m["vocab"], (blocks, c["batch"], m["k"])).astype(np.int32)
        state["forced"] = torch.from_numpy(forced).cuda()
        state["whole"] = torch.full((c["batch"],), c["k"], dtype=torch.int32, device="cuda")
    return state


def run(state):
    c, ctx = state["c"], state["ctx"]
    ctx.bpd_encode(state["src"], state["n"], state["budget"])
    if c["call"] == "encode":                      # the first proposals, and the scores of the token after the first of them
        return [ctx.bpd_get_state()[0], ctx.bpd_debug_step_logits(1)]
    if c["call"] == "steps":
        for imposed, accepted in zip(state["imposed"], state["accepted"]):
            ctx.bpd_step(c["k"], imposed, accepted)
        return [state["accepted"], *ctx.bpd_get_output()]
    if c["call"] == "scores":
        for block in state["forced"][:-1]:
            ctx.bpd_set_proposals(block)
            ctx.bpd_step(c["k"], state["whole"])
        ctx.bpd_set_proposals(state["forced"][-1])
        return ctx.bpd_debug_step_logits(c["k"])
    ids, lens, stats = ctx.bpd_decode(c["k"], state.get("schedule"))
    return [ids, lens, stats.steps, stats.accepted_total]


def _steps(c):
    return max(1, math.ceil(int(_lengths(c)[1].max()) / max(1, c["mean"])))


def work(case):
    """Steps depend on each other and a step's weights exceed what the chip keeps near its cores, so every invocation reads
    its weights once; keys and values of the prefix and of the source are read once per step and sequence."""
    c, m = case, MODELS[case["model"]]
    d, f, v, nl, k, b = m["d"], m["ff"], m["vocab"], m["layers"], c["k"], c["batch"]
    size = 4 if m["dtype"] == "f32" else 2
    n, budget = (x.astype(float) for x in _lengths(c))
    enc_w, dec_w = nl * (4 * d * d + 2 * d * f), nl * (6 * d * d + 2 * d * f)
    cross_w = nl * 2 * d * d

    def heads(count):
        return 2 * count * d * f + v * d

    # encoder, cross keys and values, first invocation with all the model's heads
    nbytes = size * (enc_w + cross_w + dec_w + heads(m["k"]) + n.sum() * d * nl * 4)
    flops = 2 * n.sum() * (enc_w + cross_w) + 4 * d * nl * float((n * n).sum()) + 2 * b * (dec_w + 2 * m["k"] * d * f + m["k"] * v * d)
    if c["call"] == "encode":
        nbytes += size * (dec_w + heads(1) + 2 * d * nl * n.sum()) + 4 * b * v
        flops += 2 * b * (dec_w + 2 * d * f + v * d)
    else:
        steps = max(1, c["target"] // k) if c["call"] == "scores" else _steps(c)
        prefix = np.minimum(budget / 2, c["local"] * 1.5) if c["local"] else budget / 2
        kv = 2 * d * nl * float((prefix + n).sum())
        rows = (2 * k - 1) if c["two_phase"] and b * k > 16 and k > 1 and size == 2 else k * k
        nbytes += steps * size * (dec_w + heads(k) + kv)
        flops += steps * (2 * b * (k * dec_w + rows * (2 * d * f + v * d)) + 2 * k * kv)
    if c["call"] == "scores":
        nbytes += 4 * b * k * k * v
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    """Tokens, lengths and counts are whole numbers; scores are sums of products of bf16 values (fp32 for the tiny model)."""
    if case["call"] not in ("scores", "encode"):
        return "exact"
    return {"rel": 1e-5 if case["model"] == "tiny" else 1e-2}
