"""The work a decode server has this library do, as cases to be timed and compared.

One pass is one call (or, for the layer cases, one decode step's four calls) through the package's public
functions, with the context, weights, caches and output buffers a server keeps between steps.  Sizes are the
library's own workloads (Step-3's attention layer: 64 query heads of dimension 256 over one key and one value head,
hidden size 7168, query rank 2048, pages of 64 tokens) and, in draw(), the ranges around them.

A case's fields:
  op      attn | query | append | out | layer
  kv      cache type: bf16, fp8 (e4m3 codes + a scale per token), fp4 (e2m1 codes + a scale per token)
  paged   cache behind a block table (permuted pages) or contiguous
  B       sequences; q_len: new tokens per sequence (1 unless several are decoded in one pass)
  ctx     longest context; ragged: the lengths are spread evenly at random over [lo, ctx] instead of all being ctx
  lens_seed   seed of those lengths (part of the case, so that its work is known)
"""
import math
import random

import torch

import paper_2507_19427_amd as mfa
from paper_2507_19427_amd import workloads as W

H, D, DM, RANK, PAGE = W.N_Q_HEADS, W.HEAD_DIM, W.D_MODEL, W.Q_RANK, W.PAGE_SIZE
KV_BYTES = {"bf16": 4 * D, "fp8": 2 * D + 8, "fp4": D + 8}          # key and value row of a token, scales included
E2M1 = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, -0., -.5, -1, -1.5, -2, -3, -4, -6], dtype=torch.float64)
TORCH_KV = {"bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn, "fp4": torch.uint8}


def _case(name, op, B, kv="bf16", ctx=0, paged=False, q_len=1, ragged=False, lo=1, lens_seed=0):
    c = {"op": op, "kv": kv, "paged": paged, "B": B, "q_len": q_len, "ctx": ctx, "ragged": ragged, "lo": lo,
         "lens_seed": lens_seed}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: a couple of short conversations, bound by launches and latency
        _case("attn_bf16_b2_ctx256", "attn", 2, "bf16", 256),
        # the benchmark workload: 64 sequences per GPU, 4K context
        _case("attn_bf16_b64_ctx4096", "attn", 64, "bf16", 4096),
        # a serving batch as it comes: lengths all over the place, paged cache
        _case("attn_bf16_paged_b128_ragged", "attn", 128, "bf16", 8192, paged=True, ragged=True, lo=1024, lens_seed=3),
        # the deployed cache type at a large batch
        _case("attn_fp8_b128_ctx8192", "attn", 128, "fp8", 8192),
        # 8-bit paged cache, an odd number of sequences of odd lengths, long contexts among them
        _case("attn_fp8_paged_b23_ragged", "attn", 23, "fp8", 20011, paged=True, ragged=True, lo=131, lens_seed=7),
        # 4-bit storage, 8-bit arithmetic
        _case("attn_fp4_b128_ctx8192", "attn", 128, "fp4", 8192),
        # multi-token decode over the deployed cache type
        _case("attn_fp8_paged_two_tokens_b64_ctx8192", "attn", 64, "fp8", 8192, paged=True, q_len=2),
        # speculative step with three drafted tokens over a bf16 cache
        _case("attn_bf16_four_tokens_b64_ctx4096", "attn", 64, "bf16", 4096, q_len=4),
        # the low-rank query path at a full batch
        _case("query_b128", "query", 128),
        # output projection of the batch of the latency table
        _case("out_proj_b64", "out", 64),
        # a whole attention layer's decode step: few sequences, bf16 cache (latency matters)
        _case("layer_bf16_b5_ctx1500", "layer", 5, "bf16", 1500, ragged=True, lo=400, lens_seed=11),
        # a whole attention layer's decode step: 64 sequences at 8K context, 8-bit paged cache
        _case("layer_fp8_paged_b64_ctx8192", "layer", 64, "fp8", 8192, paged=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choices(["attn", "layer", "query", "append", "out"], [10, 3, 3, 2, 2])[0]
    B = _log_int(rng, 1, 128)
    if op in ("query", "out"):
        return _case(None, op, B)
    kv = rng.choice(["bf16", "fp8", "fp4"])
    paged = rng.random() < 0.5
    q_len = rng.choices([1, 2, 3, 4], [7, 3, 1, 1])[0] if op == "attn" else 1
    # tokens of cache a case may hold, so that no drawn case costs more than the largest listed one
    budget = {"attn": {"bf16": 400_000, "fp8": 700_000, "fp4": 700_000}, "layer": {"bf16": 200_000, "fp8": 400_000, "fp4": 400_000},
              "append": {"bf16": 100_000, "fp8": 100_000, "fp4": 100_000}}[op][kv] // q_len
    ctx = _log_int(rng, 64, min(32768 - PAGE, max(64, budget // B)))
    ragged = rng.random() < 0.6
    return _case(None, op, B, kv, ctx, paged, q_len, ragged, 1 if rng.random() < 0.5 else max(1, ctx // 4), rng.randrange(1 << 20))


def _lens(case):
    if not case["ragged"]:
        return [case["ctx"]] * case["B"]
    r = random.Random(case["lens_seed"])
    lens = [r.randint(case["lo"], case["ctx"]) for _ in range(case["B"])]
    lens[r.randrange(case["B"])] = case["ctx"]
    return lens


def _cache_rows(gen, shape, kv):
    """Random cache rows of one tensor: (rows, scales or None), made on the GPU a few million elements at a time."""
    n = math.prod(shape)
    width = D // 2 if kv == "fp4" else D
    rows = torch.empty(n, width, dtype=TORCH_KV[kv], device="cuda")
    scales = None if kv == "bf16" else torch.empty(n, dtype=torch.float32, device="cuda")
    for i in range(0, n, 1 << 18):
        x = torch.randn(min(1 << 18, n - i), D, generator=gen, device="cuda")
        if kv == "bf16":
            rows[i:i + len(x)] = x.to(torch.bfloat16)
        else:
            quantize = W.quantize_e4m3_per_token if kv == "fp8" else W.quantize_e2m1_per_token
            rows[i:i + len(x)], scales[i:i + len(x)] = quantize(x)
    return rows.view(*shape, width), None if scales is None else scales.view(*shape)


def _make_cache(s, gen, case, filled):
    """Keys, values, scales (and block table) with room for one token more than the context."""
    room = case["ctx"] + (1 if case["op"] in ("layer", "append") else 0)
    if case["paged"]:
        blocks = (room + PAGE - 1) // PAGE
        used = [(n + 1 + PAGE - 1) // PAGE for n in _lens(case)] if case["op"] in ("layer", "append") else [(n + PAGE - 1) // PAGE for n in _lens(case)]
        n_pages = sum(used) + 16
        shape = (n_pages, PAGE)
        perm = torch.randperm(n_pages, generator=gen, device="cuda").to(torch.int32).cpu()
        table = torch.full((case["B"], blocks), -1, dtype=torch.int32)
        at = 0
        for b, n in enumerate(used):
            table[b, :n] = perm[at:at + n]
            at += n
        s["table"] = table.cuda()
    else:
        shape = (case["B"], room)
        s["table"] = None
    if filled:
        s["k"], s["ks"] = _cache_rows(gen, shape, case["kv"])
        s["v"], s["vs"] = _cache_rows(gen, shape, case["kv"])
    else:                                                     # appending reads nothing of the cache: an empty one
        width = D // 2 if case["kv"] == "fp4" else D
        for key in ("k", "v"):
            s[key] = torch.zeros(*shape, width, dtype=torch.uint8 if case["kv"] != "bf16" else torch.bfloat16, device="cuda").view(TORCH_KV[case["kv"]])
            s[key + "s"] = None if case["kv"] == "bf16" else torch.zeros(*shape, device="cuda")
    s["lens"] = torch.tensor(_lens(case), dtype=torch.int32, device="cuda")


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, std=1.0, dtype=torch.bfloat16):
        return (torch.randn(*shape, generator=gen, device="cuda") * std).to(dtype)

    op, B = case["op"], case["B"]
    s = {"case": case, "ctx": mfa.mfa_decode_init(mfa.MfaConfig())}
    if op in ("query", "append", "layer"):
        s["x"] = normal(B, DM)
    if op in ("query", "layer"):
        s["w_qa"], s["w_qb"] = normal(DM, RANK, std=0.02), normal(RANK, H * D, std=0.02)
        s["gain"] = 1.0 + normal(RANK, std=0.1, dtype=torch.float32)
        s["q"] = torch.empty(B, H, D, dtype=torch.bfloat16, device="cuda")
    if op in ("append", "layer"):
        s["w_kv"] = normal(DM, 2 * D, std=0.02)
    if op == "attn":
        s["q"] = normal(B, H, D) if case["q_len"] == 1 else normal(B, case["q_len"], H, D)
    if op in ("attn", "append", "layer"):
        _make_cache(s, gen, case, filled=op != "append")
    if op in ("attn", "layer"):
        s["out"] = torch.empty(s["q"].shape, dtype=torch.float32, device="cuda")
    if op == "layer":
        s["lens_after"] = s["lens"] + 1                       # what the attention sees: the new token included
    if op == "out":
        s["attn"] = normal(B, H, D, std=0.1, dtype=torch.float32)     # means of values: small numbers
    if op in ("out", "layer"):
        s["w_o"] = normal(H * D, DM, std=0.02)
        s["y"] = torch.empty(B, DM, dtype=torch.bfloat16, device="cuda")
    return s


def _attend(s, lens, hint, q):
    ctx, case = s["ctx"], s["case"]
    if case["paged"]:
        f = mfa.mfa_decode_attn_paged if q.dim() == 3 else mfa.mfa_decode_attn_paged_multi
        return f(ctx, q, s["k"], s["v"], s["table"], lens, hint, s["ks"], s["vs"], out=s["out"])
    f = mfa.mfa_decode_attn if q.dim() == 3 else mfa.mfa_decode_attn_multi
    return f(ctx, q, s["k"], s["v"], lens, hint, s["ks"], s["vs"], out=s["out"])


def _append(s):
    if s["case"]["paged"]:
        mfa.mfa_kv_append_paged(s["ctx"], s["x"], s["w_kv"], s["k"], s["v"], s["table"], s["lens"], s["ks"], s["vs"])
    else:
        mfa.mfa_kv_append(s["ctx"], s["x"], s["w_kv"], s["k"], s["v"], s["lens"], s["ks"], s["vs"])
    return {"k": s["k"], "v": s["v"], "k_scale": s["ks"], "v_scale": s["vs"]}


def run(s):
    case = s["case"]
    if case["op"] == "attn":
        return _attend(s, s["lens"], case["ctx"], s["q"])
    if case["op"] == "query":
        return mfa.mfa_query_proj(s["ctx"], s["x"], s["w_qa"], s["w_qb"], s["gain"], q_out=s["q"])
    if case["op"] == "append":
        return _append(s)
    if case["op"] == "out":
        return mfa.mfa_out_proj(s["ctx"], s["attn"], s["w_o"], y=s["y"])
    cache = _append(s)
    q = mfa.mfa_query_proj(s["ctx"], s["x"], s["w_qa"], s["w_qb"], s["gain"], q_out=s["q"])
    _attend(s, s["lens_after"], case["ctx"] + 1, q)
    return {"y": mfa.mfa_out_proj(s["ctx"], s["out"], s["w_o"], y=s["y"]), "cache": cache}


def work(case):
    op, B, n = case["op"], case["B"], case["q_len"]
    tokens = sum(_lens(case)) if op in ("attn", "layer") else 0
    nbytes = flops = 0
    if op in ("attn", "layer"):
        tokens += B if op == "layer" else 0
        nbytes += tokens * KV_BYTES[case["kv"]] + B * n * H * D * (2 + 4) + 4 * B
        flops += 4 * tokens * n * H * D
    if op in ("query", "layer"):
        nbytes += 2 * (DM * RANK + RANK * H * D) + B * (2 * DM + 2 * H * D) + 4 * RANK
        flops += 2 * B * (DM * RANK + RANK * H * D)
    if op in ("append", "layer"):
        nbytes += 2 * DM * 2 * D + B * (2 * DM + KV_BYTES[case["kv"]])
        flops += 2 * B * DM * 2 * D
    if op in ("out", "layer"):
        nbytes += 2 * H * D * DM + B * (4 * H * D + 2 * DM)
        flops += 2 * B * H * D * DM
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Attention: weights of 8 significant bits (2^-9 relative each, partly averaged out), sums in 32 bits.  The
    # projections round their result to bf16 (2^-9), the query path its normalised row as well.  "max" is over the
    # result's root mean square: single elements of a row whose heaviest token dominates, or of a cancelling sum.
    if case["op"] == "attn":
        return {"rel": 6e-3, "max": 5e-2}
    if case["op"] in ("query", "out"):
        return {"rel": 8e-3, "max": 5e-2}
    # Cache records: a code next to a rounding boundary may fall to either side (one step is 1/8 of an e4m3 value, half
    # of an e2m1 one), whole numbers in the packed 4-bit cache; bf16 rows differ by a rounding.
    record = {"rel": 1e-2, "max": {"bf16": 2e-2, "fp8": 0.15, "fp4": 0.15}[case["kv"]], "differ": 1e-3}
    if case["op"] == "append":
        return record
    # The layer's result adds up the query path, the attention and the output projection.
    return {"rel": 1.5e-2, "max": 0.2, "differ": 1e-3}


def _decode(rows, scales, kv):
    if kv == "fp4":
        rows = torch.stack([E2M1.cuda()[(rows & 15).long()], E2M1.cuda()[(rows >> 4).long()]], dim=-1).flatten(-2)
    else:
        rows = rows.double()
    return rows if scales is None else rows * scales.double().unsqueeze(-1)


def _exact_attention(s, lens, q):
    case = s["case"]
    q = q.double().view(case["B"], case["q_len"], H, D)
    out = torch.empty_like(q)
    for b, n in enumerate(lens):
        def rows(t, b=b, n=n):
            if t is None:
                return None
            return t[s["table"][b, :(n + PAGE - 1) // PAGE].long()].flatten(0, 1)[:n] if case["paged"] else t[b, :n]
        k = _decode(rows(s["k"]), rows(s["ks"]), case["kv"])
        v = _decode(rows(s["v"]), rows(s["vs"]), case["kv"])
        for j in range(case["q_len"]):
            m = n - (case["q_len"] - 1 - j)
            out[b, j] = torch.softmax(q[b, j] @ k[:m].T * W.SOFTMAX_SCALE, dim=-1) @ v[:m] if m > 0 else 0.0
    return out.view(s["out"].shape)


def _exact_query(s):
    c = s["x"].double() @ s["w_qa"].double()
    c = c / torch.sqrt(c.square().mean(-1, keepdim=True) + W.RMS_EPS) * s["gain"].double()
    return (c @ s["w_qb"].double()).view(-1, H, D)


def exact(case, seed):
    s = prepare(case, seed)
    if case["op"] == "attn":
        return _exact_attention(s, _lens(case), s["q"])
    if case["op"] == "query":
        return _exact_query(s)
    if case["op"] == "out":
        return s["attn"].double().view(case["B"], -1) @ s["w_o"].double()
    # the new token's rows, before any rounding to the cache's type
    kv = s["x"].double() @ s["w_kv"].double()
    if case["op"] == "append":
        got = {}
        for key, x in (("k", kv[:, :D]), ("v", kv[:, D:])):
            full = torch.zeros(*s[key].shape[:2], D, dtype=torch.float64, device="cuda")
            scale = None if case["kv"] == "bf16" else torch.zeros(*s[key].shape[:2], dtype=torch.float64, device="cuda")
            for b, n in enumerate(_lens(case)):
                at = (int(s["table"][b, n // PAGE]), n % PAGE) if case["paged"] else (b, n)
                if scale is not None:
                    scale[at] = x[b].abs().max().clamp(min=1e-12) / {"fp8": 448.0, "fp4": 6.0}[case["kv"]]
                full[at] = x[b] if scale is None else x[b] / scale[at]
            got[key] = None if case["kv"] == "fp4" else full      # (packed codes are whole numbers)
            got[key + "_scale"] = scale
        return got
    # the layer: the new rows enter the attention as the cache stores them
    for key, x in (("k", kv[:, :D]), ("v", kv[:, D:])):
        for b, n in enumerate(_lens(case)):
            at = (int(s["table"][b, n // PAGE]), n % PAGE) if case["paged"] else (b, n)
            if case["kv"] == "bf16":
                s[key][at] = x[b].to(torch.bfloat16)
                continue
            scale = x[b].float().abs().max().clamp(min=1e-12) / {"fp8": 448.0, "fp4": 6.0}[case["kv"]]
            s[key + "s"][at] = scale
            if case["kv"] == "fp8":
                s[key][at] = (x[b].float() / scale).to(torch.float8_e4m3fn)
            else:
                code = ((x[b].float() / scale).abs().unsqueeze(-1) - E2M1[:8].float().cuda()).abs().argmin(-1) + 8 * (x[b] < 0).long()
                s[key][at] = (code[0::2] | (code[1::2] << 4)).to(torch.uint8)
    s["q"] = _exact_query(s)
    a = _exact_attention(s, [n + 1 for n in _lens(case)], s["q"])
    y = a.view(case["B"], -1) @ s["w_o"].double()
    return {"y": y, "cache": {"k": None, "v": None, "k_scale": None, "v_scale": None}}
