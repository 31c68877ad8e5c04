"""The workloads whose speed matters to a user of this library: decode steps, multi-token chunks and KV transfers over a
paged cache, each through the public binding exactly as a serving loop calls it.

A case is a dict of plain values.  ``prepare`` builds what a serving engine holds before the call (pools, block table,
queries, new rows, a handle with its workspace) on the GPU, from a seed; ``run`` makes one pass.  Appends write the same
rows to the same slots on every pass, so a pass may be repeated on its state.

Context lengths are stratified over their range (every seed draws other lengths, their sum hardly moves), pages are
assigned in random order, and all values are normal with deviation one, as in ``workloads.py``.
"""
import math

import torch

from paper_2602_02204_amd import binding as omni

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
CODES = {"f32": omni.OMNI_F32, "bf16": omni.OMNI_BF16, "fp8": omni.OMNI_FP8_E4M3}
FP8_MAX = 448.0


def _decode(name, batch, heads, kv_heads, shortest, longest, **more):
    case = {"name": name, "path": "decode", "dtype": "bf16", "batch": batch, "heads": heads, "kv_heads": kv_heads,
            "head_dim": 128, "page": 16, "shortest": shortest, "longest": longest, "skewed": False, "pool": 1.0,
            "tokens": 1, "quantise": False, "out": "f32"}
    case.update(more)
    return case


def _chunks(name, batch, heads, kv_heads, shortest, longest, chunk_shortest, chunk_longest, **more):
    case = {"name": name, "path": "chunks", "dtype": "bf16", "batch": batch, "heads": heads, "kv_heads": kv_heads,
            "head_dim": 128, "page": 16, "shortest": shortest, "longest": longest, "skewed": False, "pool": 1.0,
            "chunk_shortest": chunk_shortest, "chunk_longest": chunk_longest, "out": "f32"}
    case.update(more)
    return case


def listed():
    return [
        # The smallest call: a handful of short requests over an fp32 cache (the "tiny" configuration's shape).
        _decode("tiny_f32", 4, 4, 2, 17, 200, dtype="f32", head_dim=64),
        # One user talking to a text stage: a decode step of a single request, where only latency counts.
        _decode("single", 1, 28, 4, 2048, 4096),
        # The four stage-shaped decode batches: a text stage, a speech-token stage, long multimodal prompts, and a skewed
        # mix of short and long requests in a fragmented pool of larger pages.
        _decode("thinker", 64, 28, 4, 512, 4096),
        _decode("talker", 256, 16, 2, 129, 1025),
        _decode("long", 8, 28, 4, 16384, 32768),
        _decode("mixed", 128, 32, 8, 64, 16384, page=32, skewed=True, pool=2.0),
        # The text stage over an 8-bit cache: the new bf16 rows are quantised on the device, then attended to.
        _decode("thinker_fp8", 64, 28, 4, 512, 4096, dtype="fp8", quantise=True),
        # Speculative decoding / multi-token prediction: up to two new tokens per request, their number varying.
        _decode("thinker_two_tokens", 64, 28, 4, 512, 4096, tokens=2),
        # A speech-token stage whose model has 64-dim heads: its decode step ...
        _decode("talker_d64", 256, 16, 2, 129, 1025, head_dim=64),
        # ... and its prompts: chunks of very different lengths in one call, as continuous batching mixes them.
        _chunks("chunks_ragged_d64", 24, 16, 2, 129, 2049, 1, 1024, head_dim=64, out="bf16"),
        # Chunked prefill of a text stage: 512 new tokens for each of 32 requests.
        _chunks("chunks_thinker", 32, 28, 4, 512, 4096, 512, 512),
        # The connector's payload between a prefill and a decode engine: whole requests out of one pool into another.
        {"name": "transfer", "path": "transfer", "dtype": "bf16", "batch": 64, "heads": 28, "kv_heads": 4, "head_dim": 128,
         "page": 16, "shortest": 512, "longest": 4096, "skewed": False, "pool": 1.0},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(("decode", "decode", "decode", "chunks", "chunks", "transfer"))
    # 8-bit caches exist for 128-dim heads, several tokens per decode step for the 16-bit and 8-bit caches of such heads
    dtype = rng.choice({"decode": ("bf16", "bf16", "bf16", "fp8", "f32"), "chunks": ("bf16", "bf16", "fp8"),
                        "transfer": ("bf16", "fp8")}[path])
    head_dim = 128 if dtype == "fp8" else rng.choice((64, 128, 128))
    heads, kv_heads = rng.choice(((28, 4), (16, 2), (32, 8), (4, 2), (8, 8), (16, 1), (15, 3)))
    longest = _log_uniform(rng, 64, 32768)
    shortest = max(1, int(longest * rng.choice((0.06, 0.125, 0.5, 0.9))))
    skewed = longest >= 1024 and rng.random() < 0.2
    case = {"path": path, "dtype": dtype, "batch": _log_uniform(rng, 1, 512), "heads": heads, "kv_heads": kv_heads,
            "head_dim": head_dim, "page": rng.choice((16, 16, 32)), "shortest": shortest, "longest": longest,
            "skewed": skewed, "pool": rng.choice((1.0, 1.0, 2.0))}
    if path == "decode":
        multi = dtype != "f32" and head_dim == 128 and rng.random() < 0.25
        case.update(tokens=rng.randint(2, max(2, min(8, 16 // (heads // kv_heads)))) if multi else 1,
                    quantise=dtype == "fp8" and not multi and rng.random() < 0.5,
                    out="f32" if dtype == "f32" else rng.choice(("f32", "bf16")))
    if path == "chunks":
        chunk_longest = min(longest, _log_uniform(rng, 16, 2048))
        case.update(chunk_shortest=max(1, int(chunk_longest * rng.choice((0.01, 0.25, 1.0)))), chunk_longest=chunk_longest,
                    out=rng.choice(("f32", "bf16")))
    # No more than the largest listed cases: 0.8 GB of cache per pass, and for chunks the arithmetic of theirs.
    most = {"bytes": 8e8, "flops": 4.5e11 if head_dim == 128 else 2e10}
    while case["batch"] > 1 and any(work(case)[k] > most[k] for k in most):
        case["batch"] = max(1, int(case["batch"] * 0.8))
    while path == "chunks" and work(case)["flops"] > most["flops"]:
        for key in ("longest", "shortest", "chunk_longest", "chunk_shortest"):
            case[key] = max(1, int(case[key] * 0.8))
    return case


def _strata(n, lo, hi, g=None):
    """n integers of [lo, hi] in random order, one from each n-th part of the range; without a generator the largest that
    each part holds."""
    at = torch.ones(n, dtype=torch.float64) if g is None else torch.rand(n, generator=g, dtype=torch.float64)
    x = (torch.arange(n, dtype=torch.float64) + at) / n
    got = (lo + torch.floor(x * (hi - lo + 1)).long()).clamp(max=hi)
    return got if g is None else got[torch.randperm(n, generator=g)]


def _split(case):
    """Requests drawn from the short range, from the long range, and the two ranges (a tenth is long in a skewed batch)."""
    lo, hi, n = case["shortest"], case["longest"], case["batch"]
    if not case["skewed"]:
        return (n, lo, hi), (0, lo, hi)
    n_long = int(round(0.1 * n))
    return (n - n_long, lo, min(hi, 8 * lo)), (n_long, hi // 2, hi)


def _lengths(case, g=None):
    (n0, lo0, hi0), (n1, lo1, hi1) = _split(case)
    lens = torch.cat([_strata(n0, lo0, hi0, g), _strata(n1, lo1, hi1, g)])
    return lens if g is None else lens[torch.randperm(case["batch"], generator=g)]


def _quantised(x):
    """bf16 rows [P, Hkv, page, D] -> E4M3 bytes and the scale of every (page, KV head)."""
    scale = x.abs().amax(dim=(2, 3)).float().clamp(min=1e-6) / FP8_MAX
    q = (x.float() / scale[:, :, None, None]).to(torch.float8_e4m3fn)
    return q.view(torch.uint8), scale


class State:
    pass


def prepare(case, seed):
    g = torch.Generator().manual_seed(seed)
    gd = torch.Generator(device="cuda").manual_seed(seed)
    B, Hq, Hkv, D, ps = case["batch"], case["heads"], case["kv_heads"], case["head_dim"], case["page"]
    fp8 = case["dtype"] == "fp8"
    dtype = torch.bfloat16 if fp8 else DTYPES[case["dtype"]]
    s = State()
    s.path, s.fp8, s.quantise = case["path"], fp8, bool(case.get("quantise"))

    lens = _lengths(case, g)
    pages = (lens + ps - 1) // ps
    used = int(pages.sum())
    most = _lengths(case)                        # pools and buffers are sized once, for the most a batch of the case can need
    P = int(math.ceil(int(((most + ps - 1) // ps).sum()) * case["pool"]))
    MB = (case["longest"] + ps - 1) // ps
    table = torch.full((B, MB), -1, dtype=torch.int32)
    table[torch.arange(MB)[None, :] < pages[:, None]] = torch.randperm(P, generator=g)[:used].to(torch.int32)
    s.block_table, s.context_lens = table.cuda(), lens.to(torch.int32).cuda()
    s.scale = 1.0 / math.sqrt(D)

    def normal(*shape):
        return torch.randn(shape, generator=gd, device="cuda", dtype=dtype)

    def pool():
        x = normal(P, Hkv, ps, D)
        return _quantised(x) if fp8 else (x, None)

    s.k_cache, s.k_scale = pool()
    s.v_cache, s.v_scale = pool()
    s.h = omni.Handle(batch=B, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=D, page_size=ps, num_pages=P, max_blocks_per_seq=MB,
                      kv_dtype=CODES[case["dtype"]], q_dtype=omni.OMNI_BF16 if fp8 else None,
                      out_dtype=CODES[case.get("out", "f32")])
    if s.path == "transfer":
        offsets = torch.cumsum(lens, 0) - lens
        s.token_offsets = offsets.cuda()
        s.k_dense, s.v_dense = (torch.zeros((int(most.sum()), Hkv, D), dtype=s.k_cache.dtype, device="cuda") for _ in range(2))
        s.k_other, s.v_other = torch.zeros_like(s.k_cache), torch.zeros_like(s.v_cache)
        other = torch.full((B, MB), -1, dtype=torch.int32)                   # the receiving engine's own pages
        other[table >= 0] = torch.randperm(P, generator=g)[:used].to(torch.int32)
        s.other_table = other.cuda()
        return s
    if s.path == "decode":
        s.tokens = case["tokens"]
        s.lead = (B,) if s.tokens == 1 else (B, s.tokens)
        if s.tokens > 1:
            s.h.omni_set_tuning(omni.OMNI_TUNE_QUERY_TOKENS, s.tokens)
            s.h.omni_set_query_lens(_strata(B, 1, s.tokens, g).to(torch.int32).cuda())
        s.positions = s.context_lens - 1
        s.h.alloc_workspace()
    else:
        chunk = torch.minimum(_strata(B, case["chunk_shortest"], case["chunk_longest"], g), lens)
        s.q_lens, s.q_offsets = chunk.to(torch.int32).cuda(), (torch.cumsum(chunk, 0) - chunk).cuda()
        s.max_q_len = case["chunk_longest"]
        s.lead = (int(_strata(B, case["chunk_shortest"], case["chunk_longest"]).sum()),)
        s.h.alloc_workspace(prefill_max_q_len=s.max_q_len)
    s.q = normal(*s.lead, Hq, D)
    s.k_new, s.v_new = normal(*s.lead, Hkv, D), normal(*s.lead, Hkv, D)
    if fp8 and not s.quantise:                   # rows that the program has divided by their page's scale already, about 1/100
        s.k_new, s.v_new = ((100 * x).clamp(-FP8_MAX, FP8_MAX).to(torch.float8_e4m3fn).view(torch.uint8)
                            for x in (s.k_new, s.v_new))
    s.out = torch.zeros((*s.lead, Hq, D), dtype=DTYPES[case["out"]], device="cuda")
    return s


def run(s):
    h = s.h
    if s.path == "transfer":
        h.omni_kv_pack(s.k_cache, s.v_cache, s.block_table, s.context_lens, s.token_offsets, s.k_dense, s.v_dense)
        h.omni_kv_unpack(s.k_dense, s.v_dense, s.k_other, s.v_other, s.other_table, s.context_lens, s.token_offsets)
        return {"k_dense": s.k_dense, "v_dense": s.v_dense, "k_cache": s.k_other, "v_cache": s.v_other}
    if s.path == "chunks":
        h.omni_kv_append_chunk(s.k_new, s.v_new, s.k_cache, s.v_cache, s.block_table, s.context_lens, s.q_lens, s.q_offsets,
                               s.max_q_len)
        if s.fp8:
            h.omni_paged_prefill_attn_fp8(s.q, s.k_cache, s.v_cache, s.k_scale, s.v_scale, s.block_table, s.context_lens,
                                          s.q_lens, s.q_offsets, s.max_q_len, s.scale, s.out)
        else:
            h.omni_paged_prefill_attn(s.q, s.k_cache, s.v_cache, s.block_table, s.context_lens, s.q_lens, s.q_offsets,
                                      s.max_q_len, s.scale, s.out)
    elif s.quantise:
        h.omni_kv_append_quant_fp8(s.k_new, s.v_new, s.k_cache, s.v_cache, s.k_scale, s.v_scale, s.block_table, s.positions, 1.0)
        h.omni_paged_decode_attn_fp8(s.q, s.k_cache, s.v_cache, s.k_scale, s.v_scale, s.block_table, s.context_lens, s.scale,
                                     s.out)
    elif s.fp8:
        h.omni_decode_step_fp8(s.q, s.k_new, s.v_new, s.k_cache, s.v_cache, s.k_scale, s.v_scale, s.block_table,
                               s.context_lens, s.scale, s.out)
    else:
        h.omni_decode_step(s.q, s.k_new, s.v_new, s.k_cache, s.v_cache, s.block_table, s.context_lens, s.scale, s.out)
    got = {"out": s.out, "k_cache": s.k_cache, "v_cache": s.v_cache}
    if s.quantise:
        got.update(k_scale=s.k_scale, v_scale=s.v_scale)
    return got


def work(case):
    """Every live K/V row read once, new rows and queries read and results written once; the two products' arithmetic."""
    B, Hq, Hkv, D = case["batch"], case["heads"], case["kv_heads"], case["head_dim"]
    size = {"f32": 4, "bf16": 2, "fp8": 1}[case["dtype"]]
    tokens = sum(n * 0.5 * (lo + hi) for n, lo, hi in _split(case))
    row = 2 * Hkv * D * size                                                 # a token's K and V rows
    if case["path"] == "transfer":
        return {"bytes": 4 * tokens * row, "flops": 0}                       # read and written, twice
    if case["path"] == "decode":
        new = B if case["tokens"] == 1 else B * 0.5 * (1 + case["tokens"])
        pairs = new * tokens / B
    else:
        new = min(B * 0.5 * (case["chunk_shortest"] + case["chunk_longest"]), tokens)
        pairs = new * max(tokens / B - 0.5 * new / B, 1.0)                   # causal inside the chunk
    q_size, out_size = (4 if case["dtype"] == "f32" else 2), {"f32": 4, "bf16": 2}[case["out"]]
    new_row = row * (2 if case.get("quantise") else 1)
    return {"bytes": tokens * row + new * (new_row + row) + new * Hq * D * (q_size + out_size), "flops": 4.0 * pairs * Hq * D}


def tolerance(case):
    if case["path"] == "transfer":
        return "exact"
    # Four times what the path differs by from itself in 64 bits, over these cases and fourteen drawn ones.
    if case["out"] == "bf16":
        return {"rel": 6.6e-3, "max": 2e-2}      # the result's own rounding: 1.65e-3, largest 5e-3
    if case["path"] == "chunks" and case["head_dim"] == 128:
        return {"rel": 8e-4, "max": 2e-2}        # fp16 softmax weights: 2.1e-4, largest 5.0e-3
    if case["dtype"] == "f32" or case["head_dim"] == 64:
        return {"rel": 1e-5, "max": 1e-4}        # fp32 sums
    return {"rel": 1.6e-5, "max": 2e-4}          # fp32 sums of 16-bit-pair softmax weights: 4.0e-6, largest 4.7e-5
