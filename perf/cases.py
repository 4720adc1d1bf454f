"""Performance cases of the retrieval-decode path: what a serving program has this library do.

A serving program hands a request's prompt over once per layer (`load_prefix`), then decodes token by token, every
token through every layer (`decode_step`, or the primitives it is made of where the program schedules them itself).
When a batch of requests has decoded its tokens, the next batch's prompts take its place.  A pass here is the decoding
of a few tokens through all layers of a context that such a program keeps -- or, for the `load` cases, the hand-over
of a batch of prompts and its first token.

A case is a dict: kind ("decode", "stepwise", "load"), host (KV pool in pinned host memory instead of HBM), layers,
batch, n_q, n_kv, dtype, ctx (prompt tokens per request), new_tokens (decoded per request before the next prompt),
tokens (decoded in one pass), budget / sink / window / tau (the method's parameters), rho (similarity of consecutive
queries).  Head dimension and page size are the library's only ones, 128 and 32.
"""
import math

import torch

from paper_2505_13109_amd import binding as fkv

HEAD_DIM, PAGE = 128, 32
STREAM = 32                       # decode inputs in hand: a ring of this many tokens (a new topic begins where it wraps)
OUTLIER_CHANNELS, OUTLIER_SCALE = (7, 43, 71, 101), 8.0   # keys and values have a few large channels

_BASE = dict(kind="decode", host=False, layers=1, batch=1, n_q=32, n_kv=8, dtype="bf16", ctx=4096, new_tokens=256, tokens=4,
             budget=2048, sink=512, window=512, tau=0.8, rho=0.9)


def _case(name, **kw):
    return dict(_BASE, name=name, **kw)


def listed():
    return [
        # the smallest call: one token through one layer of a short fp16 context, cache-resident; launch and latency count
        _case("one_layer_4k", dtype="fp16", budget=512, sink=32, window=32, new_tokens=64, tokens=1),
        # the ordinary one: single-request decoding of a 32-layer, 32/8-head model at 32K tokens, KV in HBM
        _case("decode_32k", layers=32, ctx=32768),
        # a larger model's layers (64/8 heads) at 64K tokens with a larger budget; 20 of its layers
        _case("decode_64k_g8", layers=20, n_q=64, ctx=65536, budget=4096, new_tokens=128),
        # long generation from a short prompt: 28/4 heads, strict threshold and drifting queries, so heads are corrected every step
        _case("generate_2k_g7", layers=28, n_q=28, n_kv=4, ctx=2048, new_tokens=2048, tau=0.9, rho=0.7),
        # a few requests of no round size: batch 7, 40/8 heads (G = 5), fp16, prompts that end inside a page
        _case("batch7_ragged", layers=8, batch=7, n_q=40, dtype="fp16", ctx=5003, new_tokens=512, budget=1024, sink=128, window=256),
        # many requests at once: the bandwidth-bound end, 32 requests of 32K tokens
        _case("batch32_32k", layers=2, batch=32, ctx=32768, new_tokens=512, tokens=8),
        # one very long context, a quarter of a million tokens
        _case("decode_256k", layers=4, ctx=262144, tokens=8),
        # the KV pool in pinned host memory: single request at 32K tokens, picked pages recalled over the host link
        _case("host_32k", host=True, layers=8, ctx=32768, new_tokens=4096, tokens=8),
        # the same with four requests of 124K tokens and queries that drift enough for half the heads to be corrected
        _case("host_batch4_124k", host=True, layers=2, batch=4, ctx=126976, new_tokens=4096, tokens=8, rho=0.8),
        # a program that schedules the primitives itself and wants the page ids and flags of every step
        _case("stepwise_16k", kind="stepwise", layers=8, ctx=16384),
        # prompts handed over after prefill, KV in HBM: two requests, lengths inside a page, then their first token
        _case("load_20k", kind="load", layers=8, batch=2, ctx=20011, new_tokens=64, tokens=1),
        # the same into the pinned host pool
        _case("load_host_16k", kind="load", host=True, layers=4, ctx=16001, new_tokens=64, tokens=1),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind, host = rng.choice([("decode", False)] * 6 + [("decode", True)] * 2 + [("stepwise", False)] * 2 + [("load", False), ("load", True)])
    n_kv = rng.choice([2, 4, 8, 8])
    n_q = n_kv * rng.randint(1, 8)
    budget, edges = rng.choice([(512, 32), (1024, 128), (1024, 192), (2048, 256), (2048, 512), (4096, 512)])
    sink, window = edges, rng.choice([edges, edges // 2 // PAGE * PAGE + PAGE])
    # what one context may hold, in cached tokens times KV heads (512 bytes each) over all layers and requests
    room = (4 if host and kind == "load" else 8 if host else 16) << 20
    ctx = _log_int(rng, 600, 131072 if host else 262144)
    new_tokens = 64 if kind == "load" else 4096 if host else rng.choice([256, 512])
    batch = _log_int(rng, 1, max(1, min(8 if host else 32, room // ((ctx + new_tokens) * n_kv))))
    layers = _log_int(rng, 1, max(1, min(8 if kind != "decode" else 32, room // ((ctx + new_tokens) * n_kv * batch))))
    tokens = 1 if kind == "load" else max(1, min(rng.randint(2, 8), 96 // layers))
    case = dict(kind=kind, host=host, layers=layers, batch=batch, n_q=n_q, n_kv=n_kv, dtype=rng.choice(["fp16", "bf16", "bf16"]),
                ctx=ctx, new_tokens=new_tokens, tokens=tokens, budget=budget, sink=sink, window=window,
                tau=rng.choice([0.8, 0.8, 0.9]), rho=rng.choice([0.93, 0.9, 0.9, 0.8, 0.7]))
    most = 0.5e9 if host else 6e9          # bytes of a pass: no more than the largest listed cases move
    while case["tokens"] > 1 and work(case)["bytes"] > most:
        case["tokens"] -= 1
    while case["layers"] > 1 and work(case)["bytes"] > most:
        case["layers"] -= 1
    return case


def _normal(shape, dtype, gen):
    return torch.randn(shape, dtype=dtype, device="cuda", generator=gen)


def _keys_or_values(shape, dtype, gen):
    x = _normal(shape, dtype, gen)
    x[..., list(OUTLIER_CHANNELS)] *= OUTLIER_SCALE
    return x


def _load(s):
    for layer, (K, V) in enumerate(s["prompt"]):
        s["kv"].load_prefix(layer, K, V)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype = torch.float16 if case["dtype"] == "fp16" else torch.bfloat16
    layers, batch, n_q, n_kv = case["layers"], case["batch"], case["n_q"], case["n_kv"]
    kv = fkv.FreeKV(n_layers=layers, batch=batch, n_q_heads=n_q, n_kv_heads=n_kv,
                    max_ctx=-(-(case["ctx"] + case["new_tokens"]) // PAGE) * PAGE, budget=case["budget"], sink=case["sink"],
                    window=case["window"], tau=case["tau"], dtype=case["dtype"],
                    placement=fkv.FKV_PLACE_HOST if case["host"] else fkv.FKV_PLACE_HBM)
    prompt = [tuple(_keys_or_values((batch, case["ctx"], n_kv, HEAD_DIM), dtype, gen) for _ in range(2)) for _ in range(layers)]
    # consecutive queries: q_t = rho q_(t-1) + sqrt(1 - rho^2) fresh
    q = [_normal((layers, batch, n_q, HEAD_DIM), torch.float32, gen)]
    for _ in range(STREAM - 1):
        q.append(case["rho"] * q[-1] + math.sqrt(1.0 - case["rho"] ** 2) * _normal(q[-1].shape, torch.float32, gen))
    q = [x.to(dtype) for x in q]
    new = [_keys_or_values((2, layers, batch, n_kv, HEAD_DIM), dtype, gen) for _ in range(STREAM)]
    out = torch.zeros((case["tokens"], layers, batch, n_q, HEAD_DIM), dtype=torch.float32, device="cuda")
    s = {"kv": kv, "kind": case["kind"], "tokens": case["tokens"], "layers": layers, "last": case["ctx"] + case["new_tokens"], "at": 0,
         "prompt": prompt, "copy": torch.cuda.Stream() if case["host"] else None,
         # what the model's projections hand over, one tensor for each token and layer
         "q": [[x[l] for l in range(layers)] for x in q], "k": [[x[0, l] for l in range(layers)] for x in new],
         "v": [[x[1, l] for l in range(layers)] for x in new],
         "out": out, "outs": [[out[t, l] for l in range(layers)] for t in range(case["tokens"])]}
    if case["kind"] == "stepwise":
        k = (case["budget"] - case["sink"] - case["window"]) // PAGE
        s["ids"] = torch.full((case["tokens"], layers, batch, n_kv, k), -1, dtype=torch.int32, device="cuda")
        s["flags"] = torch.zeros((case["tokens"], layers, batch, n_kv), dtype=torch.uint8, device="cuda")
        s["ids_of"] = [[s["ids"][t, l] for l in range(layers)] for t in range(case["tokens"])]
        s["flags_of"] = [[s["flags"][t, l] for l in range(layers)] for t in range(case["tokens"])]
    if case["kind"] != "load":
        _load(s)
    torch.cuda.synchronize()
    return s


def run(s):
    kv, copy, layers = s["kv"], s["copy"], range(s["layers"])
    if s["kind"] == "load" or kv.context_len(0) + s["tokens"] > s["last"]:
        _load(s)                          # the requests are done: the next ones' prompts
    for t in range(s["tokens"]):
        i = s["at"] % STREAM
        s["at"] += 1
        q, k, v, out = s["q"][i], s["k"][i], s["v"][i], s["outs"][t]
        if s["kind"] == "stepwise":
            ids, flags = s["ids_of"][t], s["flags_of"][t]
            for l in layers:
                kv.kv_append(l, k[l], v[l])
                kv.corr_check(l, q[l], flags[l])
                kv.page_select(l, q[l], ids[l])
                kv.sparse_decode_attn(l, q[l], out[l], use=fkv.FKV_USE_BY_FLAG)
                kv.commit(l)
        else:
            for l in layers:
                kv.decode_step(l, q[l], k[l], v[l], out[l], copy_stream=copy)
    return {"out": s["out"], "ids": s["ids"], "flags": s["flags"]} if s["kind"] == "stepwise" else s["out"]


def work(case):
    heads, group = case["batch"] * case["n_kv"], case["n_q"] // case["n_kv"]
    L = case["ctx"] + 1
    full = L // PAGE
    sink = min(case["sink"] // PAGE, full)
    window = min(case["window"] // PAGE, full - sink)
    cand = full - sink - window
    picked = min((case["budget"] - case["sink"] - case["window"]) // PAGE, cand)
    attended = (sink + window + picked) * PAGE + L % PAGE      # tokens a head attends
    row = HEAD_DIM * 2
    # a layer's step: page summaries of the candidates, keys and values of the attended tokens, the query and its
    # predecessor, the new token in and out, the output
    step = heads * (cand * 2 * row + attended * 2 * row + 2 * group * row + 4 * row + group * HEAD_DIM * 4)
    flops = heads * group * HEAD_DIM * (2 * cand + 4 * attended)
    n = case["layers"] * case["tokens"]
    total = {"bytes": n * step, "flops": n * flops}
    if case["kind"] == "load":            # keys and values in, the paged copy and its summaries out
        total["bytes"] += case["layers"] * heads * (case["ctx"] * 4 * row + -(-case["ctx"] // PAGE) * 2 * row)
    return total


def tolerance(case):
    # 16-bit inputs, fp32 accumulation, softmax weights carried to about 16 bits; page ids and flags are exact
    return {"rel": 3e-5}
