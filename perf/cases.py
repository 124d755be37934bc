"""What a user of this library has it do, as cases that can be timed.

Five kinds of work, all through the public entry points:

  step       one decoder layer of a serving step: cs_kv_append, then cs_paged_attention_mixed
             over decode tokens, prefill chunks, or both
  iteration  all layers of a step through cs_run_layers, with the safepoints of layer-wise
             preemption (the flag stays down)
  pages      whole-page checkpoint of all layers: cs_kv_ckpt_gather into a staging buffer and
             cs_kv_ckpt_restore from it into freshly allocated pages
  tokens     the same for single cached tokens: cs_kv_ckpt_gather_tokens, cs_kv_ckpt_restore_tokens
  host       a checkpoint round to the pinned host page store and back: cs_kv_ckpt_save_run,
             cs_kv_ckpt_load_run

A case is a dict of plain values; the lengths of its sequences follow from the case alone
(`lengths` seeds them), what the tensors hold and which pages they lie in from prepare()'s seed.
K, V and Q are N(0, 1), the pages of a sequence are a random permutation of the pool's.
"""
import ctypes
import math
import random

import torch

from paper_2410_01228_amd import binding as cs
from paper_2410_01228_amd import synth

#: Query heads, kv heads, head dim, layers of the model shapes.
MODELS = {
    "tiny": (4, 2, 64, 4),
    "llama8b": (32, 8, 128, 32),
    "qwen7b": (28, 4, 128, 28),
    "qwen14b": (40, 8, 128, 48),
    "llama70b": (64, 8, 128, 80),
}


def _batch(name, kind, model, decodes=0, ctx=(0, 0), spread="uniform", chunks=0, chunk=(0, 0), prior=(0, 0),
           dtype="bf16", page=16, layers=1, lengths=1):
    return {"name": name, "kind": kind, "model": model, "dtype": dtype, "page": page, "layers": layers,
            "decodes": decodes, "ctx_lo": ctx[0], "ctx_hi": ctx[1], "spread": spread,
            "chunks": chunks, "chunk_lo": chunk[0], "chunk_hi": chunk[1], "prior_lo": prior[0], "prior_hi": prior[1],
            "lengths": lengths}


def listed():
    return [
        # the smallest step: a few short requests, nothing but launches and latency
        _batch("tiny_step", "step", "tiny", 4, (17, 100), chunks=2, chunk=(32, 32), prior=(0, 48)),
        # a quiet moment online: a handful of chat requests decode
        _batch("llama8b_decode_few", "step", "llama8b", 8, (128, 2048)),
        # a full online decode batch
        _batch("llama8b_decode_256", "step", "llama8b", 256, (512, 4096)),
        # decode over the smaller of the two page sizes
        _batch("qwen7b_decode_page8", "step", "qwen7b", 64, (1024, 8192), page=8),
        # offline only: ragged prompt chunks fill the token budget
        _batch("llama8b_prefill", "step", "llama8b", chunks=3, chunk=(300, 1200), prior=(0, 8192)),
        # co-serving: online decodes and 2048 offline prefill tokens in one step
        _batch("qwen7b_mixed", "step", "qwen7b", 64, (1024, 8192), chunks=4, chunk=(512, 512), prior=(0, 16384)),
        # decodes of equal length resumed after a preemption, beside chunks, in fp16
        _batch("qwen14b_mixed_f16", "step", "qwen14b", 64, (4096, 4096), chunks=4, chunk=(256, 256), prior=(2048, 2048),
               dtype="f16"),
        # long contexts: the largest step
        _batch("llama70b_long_mixed", "step", "llama70b", 128, (2048, 32768), "log", chunks=1, chunk=(1024, 1024),
               prior=(30720, 30720)),
        # one whole iteration of a lightly loaded server: 24 decodes and a small offline chunk, all layers
        _batch("llama8b_iteration", "iteration", "llama8b", 24, (200, 3000), chunks=1, chunk=(200, 200), prior=(0, 2000),
               layers=32),
        # a checkpoint of 512 offline requests with 1 to 8 dirty pages each, and their resumption
        {"name": "qwen14b_ckpt_pages", "kind": "pages", "model": "qwen14b", "page": 16, "layers": 48, "count": 2304},
        # the tokens that 256 decoding requests generated in one step
        {"name": "qwen14b_ckpt_tokens", "kind": "tokens", "model": "qwen14b", "page": 16, "layers": 48, "count": 256},
        # the pages that a 1024-token offline chunk filled, to the host page store and back
        {"name": "qwen14b_ckpt_host", "kind": "host", "model": "qwen14b", "page": 16, "layers": 48, "count": 64},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("step", "iteration", "pages", "tokens", "host"), (12, 3, 2, 2, 1))[0]
    model = rng.choices(("tiny", "llama8b", "qwen7b", "qwen14b", "llama70b"), (1, 3, 3, 3, 3))[0]
    page = 16 if rng.random() < 0.75 else 8
    if kind in ("pages", "tokens", "host"):
        layers = rng.randint(1, MODELS[model][3]) if kind != "host" else MODELS[model][3]
        count = _log(rng, 1, {"pages": 2304, "tokens": 2048, "host": 64}[kind])
        c = {"kind": kind, "model": model, "page": page, "layers": layers, "count": count}
        while work(c)["bytes"] > {"pages": 2.9e10, "tokens": 1.0e9, "host": 8.0e8}[kind]:
            c["count"] = max(1, c["count"] // 2)
        return c
    while True:
        sides = rng.choices(("decode", "prefill", "both"), (4, 2, 4))[0]
        lo = _log(rng, 16, 8192)
        hi = _log(rng, lo, 32768)
        decodes = 0 if sides == "prefill" else _log(rng, 1, 256)
        chunks = 0 if sides == "decode" else rng.choice((1, 1, 2, 3, 4, 6))
        chunk = _log(rng, 17, 2048)
        prior = rng.choice((0, _log(rng, 16, 32768)))
        c = _batch("", kind, model, decodes, (lo, hi), rng.choice(("uniform", "log")), chunks,
                   (max(2, chunk // rng.choice((1, 1, 3))), chunk) if chunks else (0, 0), (0, prior) if chunks else (0, 0),
                   "bf16" if rng.random() < 0.75 else "f16", page,
                   MODELS[model][3] if kind == "iteration" else 1, rng.randrange(1 << 20))
        del c["name"]
        w = work(c)
        if w["bytes"] <= 5.6e9 and w["flops"] <= 1.0e12:
            return c


def _lengths(case):
    """(cached tokens, new tokens) of every sequence, the decodes (online) first."""
    r = random.Random(case["lengths"])

    def between(lo, hi, log=False):
        return min(hi, int(math.exp(r.uniform(math.log(lo), math.log(hi + 1))))) if log else r.randint(lo, hi)

    seqs = [(between(case["ctx_lo"], case["ctx_hi"], case["spread"] == "log"), 1) for _ in range(case["decodes"])]
    return seqs + [(between(case["prior_lo"], case["prior_hi"]), between(case["chunk_lo"], case["chunk_hi"]))
                   for _ in range(case["chunks"])]


def _randn(shape, gen, dtype=torch.bfloat16):
    return torch.randn(shape, generator=gen, device="cuda", dtype=dtype)


def _pool(layers, pages, hkv, d, page, gen, dtype=torch.bfloat16):
    t = torch.empty((layers, pages, 2, hkv, page * d), dtype=torch.bfloat16, device="cuda")
    t.view(dtype).normal_(generator=gen)
    return cs.Pool(t, layers, pages, hkv, d, page_size=page)


def prepare(case, seed):
    hq, hkv, d, _ = MODELS[case["model"]]
    layers, page = case["layers"], case["page"]
    cpu = torch.Generator().manual_seed(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    state = {"kind": case["kind"], "layers": layers}
    if case["kind"] in ("step", "iteration"):
        dtype = torch.float16 if case["dtype"] == "f16" else torch.bfloat16
        seqs = _lengths(case)
        b = synth.make_batch(synth.Shape(hq, hkv, d, layers, page), [c for c, _ in seqs], [q for _, q in seqs], cpu)
        batch = cs.Batch(b.block_tables, b.ctx_lens, b.cu_q_lens)
        lead = (layers,) if case["kind"] == "iteration" else ()
        state.update(
            pool=_pool(layers, b.num_pages, hkv, d, page, gen, dtype), batch=batch, hq=hq, scale=1.0 / math.sqrt(d),
            f16=dtype == torch.float16, q=_randn(lead + (b.T, hq, d), gen, dtype),
            k=_randn(lead + (b.T, hkv, d), gen, dtype), v=_randn(lead + (b.T, hkv, d), gen, dtype))
        state["out"] = torch.empty_like(state["q"])
        if case["kind"] == "iteration":
            # the preemption flag a scheduler thread would raise, looked at every fourth layer
            flag = ctypes.c_int32(0)
            online = case["decodes"]
            state.update(flag=flag, safepoint=cs.cs_safepoint(ctypes.addressof(flag), cs.POLL_FN(0), None, 4, online, 0),
                         workspace=cs.run_layers_workspace_for(batch, online, hq, hkv, d))
        else:
            state["workspace"] = cs.workspace_for(batch, hq, hkv, d)
        return state
    n = case["count"]
    pages = 2 * n + n // 4 + 8                          # some pages are in nobody's list
    pool = _pool(layers, pages, hkv, d, page, gen)
    ids = torch.randperm(pages, generator=cpu).to(torch.int32)[:2 * n]
    if case["kind"] == "tokens":                        # one token in each of n pages, of n other pages
        ids = ids * page + torch.randint(0, page, (2 * n,), generator=cpu, dtype=torch.int32)
        staging = torch.empty((layers, n, 2, hkv, d), dtype=torch.bfloat16, device="cuda")
    else:
        staging = torch.empty((layers, n, pool.page_elems) if case["kind"] == "pages" else (n, layers, pool.page_elems),
                              dtype=torch.bfloat16, device="cuda")
    state.update(pool=pool, old=ids[:n].cuda(), new=ids[n:].cuda(), staging=staging)
    if case["kind"] == "host":
        state["store"] = cs.HostStore(torch.empty((n, layers, pool.page_elems), dtype=torch.bfloat16, pin_memory=True))
    return state


def run(state):
    kind, pool, layers = state["kind"], state["pool"], state["layers"]
    if kind == "step":
        cs.cs_kv_append(pool, 0, state["batch"], state["k"], state["v"])
        attend = cs.cs_paged_attention_mixed_f16 if state["f16"] else cs.cs_paged_attention_mixed
        attend(pool, 0, state["batch"], state["q"], state["out"], state["hq"], state["scale"], state["workspace"])
        return {"out": state["out"], "pool": pool.tensor.view(torch.int16)}
    if kind == "iteration":
        first = cs.cs_run_layers(pool, 0, layers, state["batch"], state["q"], state["k"], state["v"], state["out"],
                                 state["hq"], state["scale"], state["workspace"], state["safepoint"], f16=state["f16"])
        return {"out": state["out"], "pool": pool.tensor.view(torch.int16), "preempted_before": first}
    if kind == "pages":
        cs.cs_kv_ckpt_gather(pool, 0, layers, state["old"], state["staging"])
        cs.cs_kv_ckpt_restore(pool, 0, layers, state["new"], state["staging"])
    elif kind == "tokens":
        cs.cs_kv_ckpt_gather_tokens(pool, 0, layers, state["old"], state["staging"])
        cs.cs_kv_ckpt_restore_tokens(pool, 0, layers, state["new"], state["staging"])
    else:
        cs.cs_kv_ckpt_save_run(pool, 0, layers, state["old"], state["staging"], state["store"], 0)
        cs.cs_kv_ckpt_load_run(pool, 0, layers, state["new"], state["staging"], state["store"], 0)
        return {"store": state["store"].tensor.view(torch.int16), "pool": pool.tensor.view(torch.int16)}
    return {"staging": state["staging"].view(torch.int16), "pool": pool.tensor.view(torch.int16)}


def work(case):
    hq, hkv, d, _ = MODELS[case["model"]]
    layers = case["layers"]
    if case["kind"] in ("step", "iteration"):
        nbytes = flops = 0
        for c, q in _lengths(case):
            # K/V of the sequence read once, its new tokens' K/V read once and written once, Q read and
            # the output written once, its page table read once
            nbytes += (c + q) * 2 * hkv * d * 2 + 2 * q * 2 * hkv * d * 2 + 2 * q * hq * d * 2 + 4 * -(-(c + q) // case["page"])
            flops += 4 * hq * d * (q * c + q * (q + 1) // 2)
        return {"bytes": nbytes * layers, "flops": flops * layers}
    tokens = case["count"] * (1 if case["kind"] == "tokens" else case["page"])
    # read and written on the way out, read and written on the way back (host: two of the four are
    # the host link's, which is what bounds that kind)
    return {"bytes": 4 * layers * tokens * 2 * hkv * d * 2, "flops": 0}


def tolerance(case):
    if case["kind"] not in ("step", "iteration"):
        return "exact"
    # weights and outputs are rounded to the 16-bit type (8 and 11 significant bits); what was
    # appended to the pool is bit for bit the same
    return {"rel": 1e-2, "max": 6e-2} if case["dtype"] == "bf16" else {"rel": 2e-3, "max": 2e-2}
