"""The attention and cache calls of a multimodal serving instance, as its layers make them.

Every case is one layer's share of one batch, taken through the public entry points:

  encode       bidirectional attention inside each image of a packed batch (vision encoder)
  prefill      causal attention over packed requests, and the scatter of their K/V into the paged cache
  decode       one new token per request: its K/V into the cache, then attention over the whole context
  hybrid       decode steps and chunks of prefill requests in one batch, over the paged cache
  image_cache  encoder output rows into the pages of the image cache, and back out of them

Head counts, lengths and page sizes are those of synth_inputs.py: 16 heads of 64 with 577 tokens per image and 16 heads of
80 with 256 to 4096 tokens per image (encoders); 32 / 32 heads of 128 and 28 / 4 heads of 128 (language models), requests of
an image part and a text part; cache blocks of 16 tokens, image pages of 576 rows.  Ragged lengths follow from the case
alone (`shape`), values, page tables and slots from the seed.
"""
import math
import random

import torch

import paper_2505_12658_amd as hydra

BLOCK = 16  # tokens per KV-cache block
PAGE = 576  # rows per image-cache page
CLIP_TOKENS = 577

CLIP = {"q_heads": 16, "kv_heads": 16, "head_dim": 64}
VIT = {"q_heads": 16, "kv_heads": 16, "head_dim": 80}
MHA = {"q_heads": 32, "kv_heads": 32, "head_dim": 128}
GQA = {"q_heads": 28, "kv_heads": 4, "head_dim": 128}


def listed():
    return [
        # one image of a chat request: nothing to batch it with, so the call's latency is all there is
        dict(name="encode_one_image", kind="encode", **CLIP, images=1, shape=0),
        # the encoder's usual batch: images of one fixed resolution, QKV from one fused projection
        dict(name="encode_clip_batch", kind="encode", **CLIP, images=32, shape=0),
        # the largest encoder batch: dynamic resolution, 256 to 4096 tokens per image, 64k tokens together
        dict(name="encode_vit_ragged", kind="encode", **VIT, tokens=65536, shape=0),
        # one request alone: time to first token of an idle instance
        dict(name="prefill_one_request", kind="prefill", **GQA, requests=1, prebuilt=False, shape=1),
        # prefill batch with one KV head per query head, QKV from one fused projection
        dict(name="prefill_mha_batch", kind="prefill", **MHA, requests=16, prebuilt=True, shape=0),
        # prefill batch with grouped heads: the work list built for the batch, then a layer's attention and scatter
        dict(name="prefill_gqa_batch", kind="prefill", **GQA, requests=48, prebuilt=True, shape=0),
        # a few requests being answered: the decode step between two tokens of an interactive user
        dict(name="decode_few", kind="decode", **GQA, requests=4, context_lo=300, context_hi=1500, shape=0),
        # decode of a loaded instance: contexts of a prompt and what has been generated so far
        dict(name="decode_batch", kind="decode", **GQA, requests=96, context_lo=128, context_hi=1800, shape=0),
        # the same with one KV head per query head, where the cache traffic per token is eight times as large
        dict(name="decode_mha", kind="decode", **MHA, requests=33, context_lo=600, context_hi=1100, shape=0),
        # few requests with long contexts
        dict(name="decode_long", kind="decode", **GQA, requests=8, context_lo=16384, context_hi=16384, shape=0),
        # decode steps and prefill chunks filled into one batch under a token budget
        dict(name="hybrid_batch", kind="hybrid", **GQA, requests=96, context_lo=128, context_hi=1800, chunks=4, chunk=512, shape=0),
        # an encode batch's output rows on their way through the image cache
        dict(name="image_cache_batch", kind="image_cache", hidden=3584, images=32, tokens_lo=64, tokens_hi=1024, shape=0),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["encode", "encode", "prefill", "prefill", "decode", "decode", "decode", "hybrid", "image_cache"])
    shape = rng.randrange(1 << 20)
    if kind == "encode":
        if rng.random() < 0.5:
            return dict(kind=kind, **CLIP, images=_log_int(rng, 1, 48), shape=shape)
        return dict(kind=kind, **VIT, tokens=_log_int(rng, 600, 49152), shape=shape)
    if kind == "prefill":
        heads, most = rng.choice([(MHA, 16), (GQA, 48)])
        return dict(kind=kind, **heads, requests=_log_int(rng, 1, most), prebuilt=rng.random() < 0.5, shape=shape)
    if kind == "decode":
        heads, most = rng.choice([(MHA, 32768), (GQA, 131072), (GQA, 131072)])
        hi = _log_int(rng, 200, 16384)
        lo = max(17, int(hi * rng.uniform(0.1, 0.9)))
        return dict(kind=kind, **heads, requests=_log_int(rng, 1, max(1, min(256, most // hi))), context_lo=lo, context_hi=hi, shape=shape)
    if kind == "hybrid":
        hi = _log_int(rng, 400, 2500)
        return dict(kind=kind, **GQA, requests=_log_int(rng, 4, 96), context_lo=max(17, hi // 10), context_hi=hi, chunks=rng.randint(1, 4),
                    chunk=_log_int(rng, 60, 512), shape=shape)
    hi = _log_int(rng, 64, 1024)
    return dict(kind=kind, hidden=rng.choice([3584, 4096]), images=_log_int(rng, 1, 32), tokens_lo=max(16, hi // 4), tokens_hi=hi, shape=shape)


def _lengths(case):
    """New tokens and context of every sequence of the batch (equal for encode and prefill; rows of every image)."""
    rng = random.Random(case["shape"])
    kind = case["kind"]
    if kind == "encode":
        if "images" in case:
            new = [CLIP_TOKENS] * case["images"]
        else:
            new, left = [], case["tokens"]
            while left >= 256:
                n = min(4 * (_log_int(rng, 256, 4096) // 4), left - left % 4)
                new.append(n)
                left -= n
        return new, new
    if kind == "prefill":
        if case["kv_heads"] == case["q_heads"]:
            new = [576 + rng.randint(16, 256) for _ in range(case["requests"])]
        else:
            new = [_log_int(rng, 64, 1024) + rng.randint(32, 512) for _ in range(case["requests"])]
        return new, new
    if kind == "image_cache":
        new = [_log_int(rng, case["tokens_lo"], case["tokens_hi"]) for _ in range(case["images"])]
        return new, new
    pairs = [(1, _log_int(rng, case["context_lo"], case["context_hi"])) for _ in range(case["requests"])]
    for c in range(case.get("chunks", 0)):  # chunk c of a prompt has c chunks before it in the cache
        pairs.append((case["chunk"], (c + 1) * case["chunk"]))
    rng.shuffle(pairs)
    return [n for n, _ in pairs], [c for _, c in pairs]


def _offsets(lengths):
    at, out = 0, [0]
    for n in lengths:
        at += n
        out.append(at)
    return out


def _pages(lengths, page, spare, gen, dev):
    """Pages off a shuffled free list: (pages in the cache, one row of page ids per sequence, padded with -1)."""
    need = [-(-n // page) for n in lengths]
    total = sum(need) + spare
    ids = torch.randperm(total, generator=gen, device=dev).to(torch.int32)
    width = max(need)
    column = torch.arange(width, device=dev)
    starts = torch.tensor(_offsets(need)[:-1], device=dev)
    used = column[None, :] < torch.tensor(need, device=dev)[:, None]
    at = torch.where(used, starts[:, None] + column[None, :], 0)
    return total, torch.where(used, ids[at], -1).to(torch.int32).contiguous()


def _slots(table, new, context, page, dev):
    """Cache row of each sequence's last `new` positions, one after the other."""
    counts = torch.tensor(new, device=dev)
    seq = torch.repeat_interleave(torch.arange(len(new), device=dev), counts)
    first = torch.tensor([c - n for n, c in zip(new, context)], device=dev) - torch.tensor(_offsets(new)[:-1], device=dev)
    position = torch.arange(sum(new), device=dev) + first[seq]
    return (table[seq, position // page].to(torch.int64) * page + position % page).contiguous()


def prepare(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def normal(*shape, std=1.0):
        return (torch.randn(shape, generator=gen, device=dev) * std).to(torch.bfloat16)

    new, context = _lengths(case)
    n = sum(new)
    kind = case["kind"]
    if kind == "image_cache":
        pages, table = _pages(new, PAGE, 2, gen, dev)
        rows, cache = normal(n, case["hidden"]), torch.zeros((pages, PAGE, case["hidden"]), dtype=torch.bfloat16, device=dev)
        return {"case": case, "rows": rows, "cache": cache, "slots": _slots(table, new, new, PAGE, dev), "embeddings": torch.zeros_like(rows)}

    hq, hkv, d = case["q_heads"], case["kv_heads"], case["head_dim"]
    s = {"case": case, "scale": 1.0 / math.sqrt(d), "longest": max(new)}
    if hq == hkv and kind in ("encode", "prefill") and d != 80:  # views into one projection's output
        fused = normal(n, 3 * hq * d, std=0.5 if d == 64 else 1.0)
        s["q"], s["k"], s["v"] = (fused[:, i * hq * d:(i + 1) * hq * d].view(n, hq, d) for i in range(3))
    else:
        s["q"], s["k"], s["v"] = normal(n, hq, d), normal(n, hkv, d), normal(n, hkv, d)
    s["cu"] = torch.tensor(_offsets(new), dtype=torch.int32, device=dev)
    if kind == "encode":
        return s

    blocks, s["table"] = _pages(context, BLOCK, 8, gen, dev)
    s["slots"] = _slots(s["table"], new, context, BLOCK, dev)
    s["out"] = torch.empty((n, hq, d), dtype=torch.bfloat16, device=dev)
    if kind == "prefill":
        s["k_cache"] = torch.zeros((blocks, BLOCK, hkv, d), dtype=torch.bfloat16, device=dev)
        s["v_cache"] = torch.zeros_like(s["k_cache"])
        need = hydra.hydra_attn_workspace_bytes(len(new), n, s["longest"], hq, hkv, d)
    else:
        s["k_cache"], s["v_cache"] = normal(blocks, BLOCK, hkv, d), normal(blocks, BLOCK, hkv, d)
        s["kv_lens"] = torch.tensor(context, dtype=torch.int32, device=dev)
        need = hydra.hydra_attn_paged_workspace_bytes(len(new), hkv, d, s["table"].shape[1], BLOCK)
    s["workspace"] = torch.empty(max(need, 16), dtype=torch.uint8, device=dev)
    # the caches' bits, as whole numbers: they are copied, not computed
    s["k_bits"], s["v_bits"] = s["k_cache"].view(torch.int16), s["v_cache"].view(torch.int16)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "encode":
        return hydra.hydra_attn_varlen_fwd(s["q"], s["k"], s["v"], s["cu"], s["longest"], False, s["scale"])
    if kind == "prefill":
        if case["prebuilt"]:
            n, hq, d = s["q"].shape
            hydra.hydra_attn_build_worklist(s["cu"], n, s["longest"], hq, case["kv_heads"], d, True, s["workspace"])
            hydra.hydra_attn_varlen_fwd_prebuilt(s["q"], s["k"], s["v"], s["cu"], s["longest"], True, s["scale"], s["out"], s["workspace"])
        else:
            hydra.hydra_attn_varlen_fwd(s["q"], s["k"], s["v"], s["cu"], s["longest"], True, s["scale"], out=s["out"], workspace=s["workspace"])
        hydra.hydra_kv_cache_write(s["k"], s["v"], s["k_cache"], s["v_cache"], s["slots"])
        return s["out"], s["k_bits"], s["v_bits"]
    if kind == "image_cache":
        hydra.hydra_page_cache_write(s["rows"], s["cache"], s["slots"])
        hydra.hydra_page_cache_gather(s["cache"], s["slots"], s["embeddings"])
        return s["cache"], s["embeddings"]
    hydra.hydra_kv_cache_write(s["k"], s["v"], s["k_cache"], s["v_cache"], s["slots"])
    hydra.hydra_attn_paged_fwd(s["q"], s["k_cache"], s["v_cache"], s["table"], s["cu"], s["kv_lens"], s["longest"], s["scale"], out=s["out"],
                               workspace=s["workspace"])
    return s["out"], s["k_bits"], s["v_bits"]


def work(case):
    new, context = _lengths(case)
    n = sum(new)
    if case["kind"] == "image_cache":  # each row read and written in both directions, and its slot
        return {"bytes": 2 * n * (2 * case["hidden"] * 2 + 8), "flops": 0}
    hq, hkv, d = case["q_heads"], case["kv_heads"], case["head_dim"]
    row = hkv * d * 2
    if case["kind"] == "encode":
        pairs = sum(L * L for L in new)
        cache = 0
    else:
        pairs = sum(q * (c - q) + q * (q + 1) // 2 for q, c in zip(new, context))
        cache = n * (2 * row + 8)  # the new tokens' rows into the cache
    old = sum(c - q for q, c in zip(new, context))  # context that only the cache holds
    return {"bytes": 2 * n * hq * d * 2 + 2 * n * row + cache + 2 * old * row, "flops": 4 * d * hq * pairs}


def tolerance(case):
    # bf16 probabilities and bf16 outputs (half a unit of 8 bits each); copies are exact
    return "exact" if case["kind"] == "image_cache" else {"rel": 1e-2}
