"""What a program built on this library has it do, as timed cases.

A case is one layer's worth of work in one of the situations the library is used in: the hooked
attention call on decode rows, on prompts, on a mixed serving step, over 16-bit and 8-bit caches, the
re-ranker's span pass with its reduction, and steering.  Calls go through the Python binding the way a
program uses it: inputs, output buffers and workspace are made once and kept, the call object is
launched once per pass on the current stream.

    listed()          the named cases
    draw(rng)         one more case of the same ranges
    prepare(case, s)  inputs and the kept call object, from the seed `s` alone
    run(state)        one pass, returning every output
    work(case)        bytes and operations the pass cannot do without
    tolerance(case)   how far another correct implementation may be off

Sequence lengths belong to the case (they come from its own `lens` number), values to the seed: queries,
keys and values are N(0, 1), which gives attention logits of unit spread.
"""
import dataclasses
import math
import random

import torch

from paper_2603_06588_amd import binding, workloads

KIND = {"decode": binding.BATCH_DECODE_ONLY, "prefill": binding.BATCH_PREFILL_ONLY, "mixed": binding.BATCH_MIXED}
E4M3_MAX = 448.0
E4M3_SIGMAS = 5.0     # an 8-bit cache's scale maps this many standard deviations to the format's largest number


def attention(name, what, n, lo, hi, **more):
    """n sequences with contexts of lo..hi tokens; `what`: decode (one row each), prefill (the whole context is
    new, or all but `prior` tokens of it) or mixed (n decode rows, then `chunks` prompts of `chunk` tokens)."""
    c = {"name": name, "path": "attention", "what": what, "n": n, "lo": lo, "hi": hi, "lens": 1, "prior": 0, "chunks": 0,
         "chunk": 0, "hq": 32, "hkv": 8, "d": 128, "dtype": "bf16", "kv8": False, "write": False, "probed": 8, "rows": 1,
         "spans": 1, "span": 256, "steer": "", "hidden": 0, "hidden_rows": 0}
    c.update(more)
    return c


def rerank(name, prompts, docs_lo, docs_hi, doc_lo, doc_hi, **more):
    c = {"name": name, "path": "rerank", "prompts": prompts, "docs_lo": docs_lo, "docs_hi": docs_hi, "doc_lo": doc_lo,
         "doc_hi": doc_hi, "question": 32, "lens": 1, "hq": 32, "hkv": 8, "d": 128, "probed": 8}
    c.update(more)
    return c


def listed():
    return [
        # a full-precision check run on a small model: every head probed at the last token, one span, and a
        # steering vector added to the last rows
        attention("tiny_fp32", "prefill", 1, 256, 256, hq=8, hkv=8, d=64, dtype="f32", probed=8, span=48, steer="add", hidden=512,
                  hidden_rows=256),
        # one conversation generating its next token: nothing but latency; the call also stores the token's key and value
        attention("decode_one", "decode", 1, 1237, 1237, write=True),
        # a lightly loaded server's decode step
        attention("decode_few", "decode", 8, 2500, 4096, write=True),
        # a full server's decode step, every head watched on the instruction part of its prompt
        attention("decode_many", "decode", 256, 1024, 8192, probed=32, span=272),
        # the same over an 8-bit cache
        attention("decode_many_kv8", "decode", 256, 1024, 8192, probed=32, span=272, kv8=True),
        # one prompt checked for injection: last token, instruction range and data range
        attention("prompt_one", "prefill", 1, 2048, 2048, spans=2),
        # a batch of ragged prompts
        attention("prefill_ragged", "prefill", 16, 512, 2048, probed=12, rows=8, span=160),
        # one long retrieval prompt on a wide model, four documents watched from the question's rows
        attention("prefill_long", "prefill", 1, 32768, 32768, hq=64, probed=16, rows=32, spans=4, span=1024),
        # chunked prefill over an 8-bit cache: the chunk's rows are quantised into the cache by the call
        attention("prefill_kv8", "prefill", 8, 1100, 3000, prior=1024, kv8=True, write=True, rows=8, span=160),
        # a small model's head size
        attention("prefill_d64", "prefill", 16, 512, 2048, d=64, probed=12, rows=8, span=160),
        # a serving step with decode rows and prompt chunks in one batch, and steering of the prompt rows afterwards
        attention("mixed_step", "mixed", 64, 4096, 4096, chunks=4, chunk=2048, write=True, steer="add", hidden=4096, hidden_rows=8448),
        # re-ranking: the question rows' attention on every document of the prompts, reduced to a score per document
        rerank("rerank", 4, 40, 100, 64, 256),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fp32", "decode", "decode", "decode", "decode", "prompt", "prefill", "prefill", "long", "prefill_kv8",
                       "prefill_d64", "mixed", "rerank"])
    lens = rng.randrange(1 << 20)
    span = _log(rng, 16, 512)
    if kind == "rerank":
        d_lo, k_lo = rng.randint(20, 64), _log(rng, 8, 60)
        c = rerank("", rng.randint(1, 4), k_lo, k_lo + rng.randint(0, 40), d_lo, d_lo + rng.randint(0, 192), lens=lens,
                   question=rng.randint(5, 48), probed=rng.randint(1, 12))
    elif kind == "fp32":
        L = _log(rng, 33, 512)
        c = attention("", "prefill", rng.randint(1, 3), L, L, lens=lens, hq=8, hkv=8, d=64, dtype="f32", probed=rng.randint(1, 8),
                      span=span, steer="add", hidden=128 * rng.randint(2, 8), hidden_rows=0)
    elif kind == "decode":
        n = _log(rng, 1, 256)
        hi = _log(rng, 128, 8192 if n > 16 else 16384)
        lo = max(64, int(hi * rng.uniform(0.12, 1.0)))
        c = attention("", "decode", n, lo, hi, lens=lens, hq=rng.choice([32, 32, 64]), kv8=rng.random() < 0.4, d=rng.choice([128, 128, 128, 64]),
                      probed=_log(rng, 1, 32), span=span, write=n * hi <= 300000 and rng.random() < 0.7)
    elif kind == "prompt":
        L = _log(rng, 65, 8192)
        c = attention("", "prefill", 1, L, L, lens=lens, probed=rng.randint(1, 16), spans=rng.randint(1, 4), span=span)
    elif kind == "long":
        L = _log(rng, 8192, 32000)
        c = attention("", "prefill", 1, L, L, lens=lens, hq=64, probed=rng.randint(4, 16), rows=rng.randint(1, 32),
                      spans=rng.randint(1, 4), span=_log(rng, 128, 1024))
    elif kind == "mixed":
        n, hi = _log(rng, 4, 96), _log(rng, 512, 6000)
        chunks, chunk = rng.randint(1, 4), _log(rng, 130, 2048)
        c = attention("", "mixed", n, max(64, int(hi * rng.uniform(0.3, 1.0))), hi, lens=lens, chunks=chunks, chunk=chunk,
                      kv8=rng.random() < 0.25, write=rng.random() < 0.7, span=span, probed=rng.randint(1, 16),
                      steer=rng.choice(["add", "fold"]), hidden=4096, hidden_rows=0)
    else:
        n, hi = rng.randint(2, 16), _log(rng, 150, 3000)
        c = attention("", "prefill", n, max(64, int(hi * rng.uniform(0.25, 1.0))), hi, lens=lens, d=64 if kind == "prefill_d64" else 128,
                      kv8=kind == "prefill_kv8", prior=rng.choice([0, 0, rng.randint(1, 2000)]), probed=rng.randint(1, 16), rows=rng.randint(1, 16),
                      spans=rng.randint(1, 3), span=span)
        c["write"] = c["kv8"]
        c["lo"], c["hi"] = c["lo"] + c["prior"], c["hi"] + c["prior"]
    del c["name"]
    return c


# ---- shapes -------------------------------------------------------------------------------------------------

def _lengths(case):
    """(contexts, new rows) of an attention case's sequences."""
    r = random.Random(case["lens"])
    ctx = [r.randint(case["lo"], case["hi"]) for _ in range(case["n"])]
    if case["what"] == "prefill":
        return ctx, [L - case["prior"] for L in ctx]
    return ctx + [case["chunk"]] * case["chunks"], [1] * case["n"] + [case["chunk"]] * case["chunks"]


def _documents(case):
    """One list of document lengths per prompt."""
    r = random.Random(case["lens"])
    return [[r.randint(case["doc_lo"], case["doc_hi"]) for _ in range(r.randint(case["docs_lo"], case["docs_hi"]))]
            for _ in range(case["prompts"])]


def _heads(case):
    return sorted({i * case["hq"] // case["probed"] for i in range(case["probed"])})


def _hidden_rows(case, total_q):
    return max(case["hidden_rows"], total_q)


# ---- inputs -------------------------------------------------------------------------------------------------

def _spans(r, L, count, length):
    """`count` disjoint ranges of about `length` keys, one in each equal part of the context."""
    part = L // count
    out = []
    for i in range(count):
        n = max(1, min(length, part))
        a = i * part + r.randint(0, part - n)
        out.append((a, a + n))
    return out


def _to_e4m3(x):
    """Bytes of a cache whose scale maps E4M3_SIGMAS standard deviations to the largest number of the format."""
    out = torch.empty(x.shape, dtype=torch.uint8, device=x.device)
    for r in range(0, x.shape[0], 4096):
        y = (x[r:r + 4096].float() * (E4M3_MAX / E4M3_SIGMAS)).clamp_(-E4M3_MAX, E4M3_MAX)
        out[r:r + 4096] = y.to(torch.float8_e4m3fn).view(torch.uint8)
    return out


def _batch(case, seed, lens, rows, query_sel, key_spans):
    gen = torch.Generator().manual_seed(seed)
    b = workloads.build_paged("case", lens, rows, case["hq"], case["hkv"], case["d"],
                              torch.float32 if case.get("dtype") == "f32" else torch.bfloat16, 1.0, gen, _heads(case), query_sel,
                              key_spans, poison=False, device="cuda", seed=seed)
    if case.get("kv8"):
        scale = torch.linspace(1.0, 1.25, case["hkv"], device="cuda") * (E4M3_SIGMAS / E4M3_MAX)
        b = dataclasses.replace(b, k_cache=_to_e4m3(b.k_cache), v_cache=_to_e4m3(b.v_cache), k_scale=scale, v_scale=scale.clone())
    return b


def prepare(case, seed):
    r = random.Random(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["path"] == "rerank":
        docs = _documents(case)
        lens, key_spans = [], []
        for d in docs:
            pos, sp = 64, []            # a 64-token preamble, the documents, the question
            for n in d:
                sp.append((pos, pos + n))
                pos += n
            key_spans.append(sp)
            lens.append(pos + case["question"])
        b = _batch(case, seed, lens, lens, [(L - case["question"], L) for L in lens], key_spans)
        P, NQ, S = len(_heads(case)), b.max_sel_q, b.max_spans
        s = {"path": "rerank", "b": b, "mass": torch.empty((len(lens), P, NQ, S), dtype=torch.float32, device="cuda"),
             "scores": torch.empty((len(lens), S), dtype=torch.float32, device="cuda"),
             "weights": torch.rand(P, generator=gen, device="cuda") + 0.5}
        # scratch for the split form of the pass: (max, sum) pairs of up to 16 key splits
        s["scratch"] = torch.empty(max(256, len(lens) * P * (NQ + 15) // 16 * 16 * 16 * 8), dtype=torch.uint8, device="cuda")
        return s
    lens, rows = _lengths(case)
    sel = [(max(0, n - case["rows"]), n) for n in rows]
    b = _batch(case, seed, lens, rows, sel, [_spans(r, L, case["spans"], case["span"]) for L in lens])
    more = {}
    if case["write"]:
        shape = (b.total_q, case["hkv"], case["d"])
        more = {"k_new": torch.randn(shape, generator=gen, device="cuda").to(b.q.dtype),
                "v_new": torch.randn(shape, generator=gen, device="cuda").to(b.q.dtype)}
    s = {"path": "attention", "b": b, "call": binding.call_from_batch(b, batch_kind=KIND[case["what"]], **more), "write": case["write"],
         "steer": case["steer"]}
    if case["steer"]:
        T, D = _hidden_rows(case, b.total_q), case["hidden"]
        s["hidden"] = torch.randn((T, D), generator=gen, device="cuda").to(b.q.dtype)
        v = torch.randn(D, generator=gen, device="cuda")
        s["vec"] = (v / v.norm()).to(b.q.dtype)
        s["mask"] = torch.zeros(T, dtype=torch.uint8, device="cuda")
        first = case["n"] if case["what"] == "mixed" else b.total_q - b.total_q // 4
        s["mask"][first:b.total_q] = 1
        if case["steer"] == "fold":
            s["delta"] = torch.randn((T, D), generator=gen, device="cuda").to(b.q.dtype)
    return s


def run(s):
    b = s["b"]
    if s["path"] == "rerank":
        binding.hook_span_mass_batch(b, mass=s["mass"], workspace=s["scratch"])
        binding.hook_reduce_mass(s["mass"], binding.REDUCE_SPAN_MEAN, query_sel=b.query_sel, cu_q_lens=b.cu_q_lens,
                                 head_weights=s["weights"], scores=s["scores"])
        return {"mass": s["mass"], "scores": s["scores"]}
    call = s["call"]
    call.launch()
    out = {"out": call.out, "mass": call.mass}
    if s["write"]:
        out["k_cache"], out["v_cache"] = b.k_cache, b.v_cache
    if s["steer"] == "fold":
        out["hidden"] = binding.hook_residual_add_steer(s["hidden"], s["delta"], s["vec"], 8.0, s["mask"])
    elif s["steer"]:
        out["hidden"] = binding.hook_steer(s["hidden"], s["vec"], 8.0, s["mask"])
    return out


# ---- what a pass cannot do without --------------------------------------------------------------------------

def work(case):
    heads = _heads(case)
    d, hkv = case["d"], case["hkv"]
    if case["path"] == "rerank":
        docs, q = _documents(case), case["question"]
        S = max(len(x) for x in docs)
        groups = len({h // (case["hq"] // hkv) for h in heads})
        keys = sum(64 + sum(x) + q for x in docs)
        pairs = sum(q * (64 + sum(x)) + q * (q + 1) // 2 for x in docs)
        out = len(docs) * S * (len(heads) * q + 1) * 4
        return {"bytes": keys * groups * d * 2 + len(docs) * q * len(heads) * d * 2 + out, "flops": 2 * d * len(heads) * pairs}
    lens, rows = _lengths(case)
    e = 4 if case["dtype"] == "f32" else 2
    ek = 1 if case["kv8"] else e
    total_q = sum(rows)
    pairs = sum(n * (L - n) + n * (n + 1) // 2 for L, n in zip(lens, rows))
    n_bytes = 2 * total_q * case["hq"] * d * e + 2 * sum(lens) * hkv * d * ek
    n_bytes += len(lens) * len(heads) * min(case["rows"], max(rows)) * case["spans"] * 4
    if case["write"]:
        n_bytes += 2 * total_q * hkv * d * e      # the new rows come from their own buffers; the cache rows they fill are counted above
    if case["steer"]:
        T, D = _hidden_rows(case, total_q), case["hidden"]
        masked = sum(rows[case["n"]:]) if case["what"] == "mixed" else total_q // 4
        n_bytes += (3 * T if case["steer"] == "fold" else 2 * masked) * D * e
    return {"bytes": n_bytes, "flops": 4 * d * case["hq"] * pairs}


def tolerance(case):
    if case["path"] == "rerank" or case["dtype"] == "f32":
        return {"rel": 2e-5, "max": 4e-4}         # fp32 sums, and exponentials of logits rounded to fp32
    return {"rel": 1e-2, "max": 0.15}             # probabilities and outputs are rounded to bf16
