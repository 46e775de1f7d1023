"""The conversion work of a serving deployment, as cases that can be timed.

A case is one transfer: the model's KV shape, the two sides' parallel
strategies, element types, storage orders and page sizes, the requests whose
KV moves, and the entry point that moves it:

    repack       kvx_repack, or kvx_repack_paged for a paged source
    noalloc      kvx_repack_noalloc (no plan, no allocation)
    pack         kvx_pack / kvx_pack_paged
    pack_unpack  the two-step path: kvx_pack(_paged), then kvx_unpack
    pipe         kvx_pipe_run, the layer-streamed transfer through host memory

`prepare` makes what a prefill and a decode engine hold before the call (KV
buffers, block tables, pools, the plan), `run` is the call, `exact` the same
result in 64 bits from plain torch.  Every result of the library is fully
specified down to its bits (copies, correctly rounded casts, codes of a
correctly rounded quotient), so outputs are compared exactly.
"""
from __future__ import annotations

import random

import torch

import paper_2509_17542_amd as K

TORCH = {"fp16": torch.float16, "bf16": torch.bfloat16}
CODE = {"fp16": K.FP16, "bf16": K.BF16, "e4m3fn": K.E4M3FN, "e5m2": K.E5M2}
ORDER = {"thd": K.THD, "htd": K.HTD, "paged": K.PAGED}
FMAX = {"e4m3fn": 448.0, "e5m2": 57344.0}


def make_case(name, op, layers, heads, dim, src_tp, dst_tp, rank, src, wire, cache, order, page,
              requests, lo, hi, lens, src_page=0, chunk=0, slots=0):
    """`wire` is the transfer type, `cache` the decode cache's; `lens` seeds
    the request lengths lo..hi, so that they belong to the case."""
    c = dict(op=op, layers=layers, heads=heads, dim=dim, src_tp=src_tp, dst_tp=dst_tp, rank=rank,
             src=src, wire=wire, cache=cache, order=order, page=page, requests=requests, lo=lo,
             hi=hi, lens=lens, src_page=src_page, chunk=chunk, slots=slots)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call: one short prompt of a tiny model, TP1 -> TP2;
        # what it costs is launching
        make_case("tiny_one_request", "repack", 2, 4, 64, 1, 2, 0, "fp16", "bf16", "bf16", "thd",
                  16, 1, 256, 256, 1),
        # steady traffic into a running decode engine that cannot allocate: a
        # batch of short chat turns, TP1 -> one rank of TP4
        make_case("chat_batch_noalloc", "noalloc", 32, 8, 128, 1, 4, 2, "bf16", "bf16", "bf16",
                  "thd", 16, 64, 16, 512, 2),
        # the ordinary call: one finished prompt of a Llama-3-8B-shaped model
        # moves as soon as its prefill ends
        make_case("llama8b_one_request", "repack", 32, 8, 128, 1, 1, 0, "bf16", "bf16", "bf16",
                  "thd", 16, 1, 1900, 1900, 3),
        # the largest: a batch of prompts of the same model
        make_case("llama8b_batch", "repack", 32, 8, 128, 1, 1, 0, "bf16", "bf16", "bf16", "thd",
                  16, 8, 512, 4096, 4),
        # both ends of a link: a Llama-3-70B shard, prefill TP4 merged into
        # decode TP2, packed into the transfer tensor and unpacked from it
        make_case("llama70b_tp4to2_pack_unpack", "pack_unpack", 80, 8, 128, 4, 2, 0, "bf16", "bf16",
                  "bf16", "thd", 32, 2, 1024, 4096, 5),
        # head-major fp16 KV with outliers into a bf16 cache of large pages
        # (Qwen-7B-style GQA), ragged last pages
        make_case("qwen_htd_fp16_bf16", "repack", 28, 4, 128, 1, 1, 0, "fp16", "bf16", "bf16", "htd",
                  64, 16, 128, 2048, 6),
        # an fp8 decode cache, one group of 4 layers: long and short prompts
        make_case("fp8_decode_group", "repack", 4, 8, 128, 1, 1, 0, "bf16", "e4m3fn", "e4m3fn", "thd",
                  16, 16, 256, 16384, 7),
        # an fp8 cache under wide tensor parallelism: one head per decode rank,
        # split from prefill TP4 shards of two heads
        make_case("llama70b_tp4to8_fp8", "repack", 80, 8, 128, 4, 8, 3, "bf16", "e4m3fn", "e4m3fn",
                  "thd", 16, 4, 512, 4096, 8),
        # a halved link: e5m2 codes and scales in the transfer tensor, from the
        # prefill side's own pages, dequantised into a bf16 cache
        make_case("e5m2_link_paged_to_bf16", "pack_unpack", 32, 8, 128, 1, 1, 0, "bf16", "e5m2",
                  "bf16", "paged", 16, 2, 512, 4096, 9, src_page=16),
        # paged to paged with a TP merge: 16-token prefill pages, 64-token
        # decode pages
        make_case("llama70b_paged16to64_tp4to2", "repack", 80, 8, 128, 4, 2, 1, "bf16", "bf16",
                  "bf16", "paged", 64, 3, 512, 4096, 10, src_page=16),
        # odd sizes: head_dim 80, six heads from TP2 to TP3 (ranks straddle
        # shards), token-granular (one-token) decode pages
        make_case("hd80_tp2to3_token_pages", "repack", 32, 6, 80, 2, 3, 1, "fp16", "bf16", "bf16",
                  "thd", 1, 5, 100, 1500, 11),
        # the layer-streamed transfer of one prompt through pinned host memory
        make_case("llama8b_layer_stream", "pipe", 32, 8, 128, 1, 1, 0, "bf16", "bf16", "bf16", "thd",
                  16, 1, 2000, 2000, 12, chunk=4, slots=3),
    ]


def draw(rng: random.Random):
    """A transfer of the same ranges: shapes of the models above and of the
    test suite (head_dim 64..256, 1..8 KV heads in all, every TP degree that
    divides them, page sizes from token-granular to 128, odd ones among
    them), every pair of types, each storage order, from one short request to
    batches; the source KV stays below the largest listed case's."""
    op = rng.choice(["repack"] * 5 + ["noalloc"] * 2 + ["pack_unpack"] * 2 + ["pack"] * 2)
    heads = rng.choice([1, 2, 4, 6, 8, 8, 8])
    dim = rng.choice([64, 80, 96, 112, 128, 128, 128, 192, 256])
    tps = [t for t in (1, 2, 3, 4, 6, 8) if heads % t == 0]
    src_tp = rng.choice(tps)
    dst_tp = rng.choice(tps + [2 * heads])      # more ranks than heads: replicated heads
    rank = rng.randrange(dst_tp)
    src = rng.choice(["bf16", "bf16", "fp16"])
    wire = rng.choice([src, "bf16", "fp16", "e4m3fn", "e4m3fn", "e5m2"])
    cache = wire
    if wire in FMAX and rng.random() < 0.4:
        cache = rng.choice(["bf16", "fp16"])
    order = rng.choice(["thd", "thd", "htd"] + (["paged"] if op != "noalloc" else []))
    page = rng.choice([1, 5, 8, 16, 16, 16, 24, 32, 64, 128])
    src_page = rng.choice([1, 16, 16, 24, 32, 64]) if order == "paged" else 0
    layers = rng.choice([4, 16, 28, 32, 48, 61, 80])
    hs, hd = heads // src_tp, max(1, heads // dst_tp)
    # source bytes the rank's heads hold: from 1 MB to 1.5 GB, spread over the logarithm
    per_token = 2 * layers * max(hs, hd) * dim * 2
    tokens = max(4, int(10 ** rng.uniform(6.0, 9.17)) // per_token)
    # what the library takes: at most 2^24 work units, 65536 pages without a
    # plan; the bound here is a quarter of the first
    pages_max = min((1 << 22) // (2 * layers * hd), 65536 if op == "noalloc" else 1 << 20)
    tokens = min(tokens, pages_max * page * 3 // 4, 200_000)
    requests = min(rng.choice([1, 1, 2, 3, 8, 17, 64, 200]), max(1, tokens // 16))
    mean = max(1, tokens // requests)
    lo, hi = (mean, mean) if requests == 1 else (max(1, mean // 4), max(1, mean + mean * 3 // 4))
    return make_case(None, op, layers, heads, dim, src_tp, dst_tp, rank, src, wire, cache, order, page,
                     requests, lo, hi, rng.randrange(1 << 30), src_page)


def lengths(c):
    r = random.Random(c["lens"])
    return [r.randint(c["lo"], c["hi"]) for _ in range(c["requests"])]


def _heads(c):
    """Heads per prefill shard and per decode rank."""
    H = c["heads"]
    return (H // c["src_tp"] if c["src_tp"] <= H else 1,
            H // c["dst_tp"] if c["dst_tp"] <= H else 1)


def _rank_heads(c):
    """(prefill shard, head within it) of each of the decode rank's heads."""
    H, (hs, hd) = c["heads"], _heads(c)
    g0 = c["rank"] * hd if c["dst_tp"] <= H else c["rank"] // (c["dst_tp"] // H)
    return [((g0 + i) // hs, (g0 + i) % hs) for i in range(hd)]


def _pages(lens, page):
    return [(t + page - 1) // page for t in lens]


def _table(lens, page, gen):
    """Pages drawn at random from a pool of twice the pages that are needed
    -> (int32 [requests, stride] on the device, pages in the pool)."""
    need = _pages(lens, page)
    pool = 2 * sum(need) + 8
    perm = torch.randperm(pool, generator=gen)
    table = torch.full((len(lens), max(need)), -1, dtype=torch.int32)
    at = 0
    for r, n in enumerate(need):
        table[r, :n] = perm[at:at + n].to(torch.int32)
        at += n
    return table.cuda(), pool


def _values(shape, head_axis, c, gen):
    """KV values: normal, every (layer, k/v, head) with a magnitude of its own
    over two decades; fp16 sources carry 0.1% outliers of +-60000."""
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    scale_shape = [1] * len(shape)
    scale_shape[0], scale_shape[head_axis] = shape[0], shape[head_axis]
    x *= 10.0 ** (2.0 * torch.rand(scale_shape, generator=gen, device="cuda") - 1.0)
    if c["src"] == "fp16":
        u = torch.rand(shape, generator=gen, device="cuda", dtype=torch.float32)
        x = torch.where(u < 0.0005, -60000.0, torch.where(u > 0.9995, 60000.0, x))
    return x.to(TORCH[c["src"]])


def _inputs(c, seed):
    """Source shards (those that the rank reads; the others None), the decode
    and the source block table."""
    lens = lengths(c)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    hgen = torch.Generator().manual_seed(seed)
    hs, _ = _heads(c)
    P, D = 2 * c["layers"], c["dim"]
    bt, pool = _table(lens, c["page"], hgen)
    sbt, spool = _table(lens, c["src_page"], hgen) if c["order"] == "paged" else (None, 0)
    shards = [None] * c["src_tp"]
    for j in sorted({j for j, _ in _rank_heads(c)}):
        if c["order"] == "paged":       # [plane][page][slot][head][dim]; a plane pair at a time
            shards[j] = torch.empty((P, spool, c["src_page"], hs, D), dtype=TORCH[c["src"]],
                                    device="cuda")
            for p in range(0, P, 2):
                shards[j][p:p + 2] = _values((2, spool, c["src_page"], hs, D), 3, c, gen)
        else:                           # requests back to back
            shards[j] = torch.empty(P * sum(lens) * hs * D, dtype=TORCH[c["src"]], device="cuda")
            at = 0
            for T in lens:
                shape, axis = ((P, T, hs, D), 2) if c["order"] == "thd" else ((P, hs, T, D), 1)
                n = P * T * hs * D
                shards[j][at:at + n] = _values(shape, axis, c, gen).reshape(-1)
                at += n
    return lens, shards, bt, pool, sbt, spool


def prepare(case, seed):
    c = case
    lens, shards, bt, pool, sbt, spool = _inputs(c, seed)
    _, hd = _heads(c)
    cache8 = c["cache"] in FMAX
    desc = K.make_desc(c["layers"], c["heads"], c["dim"], c["src_tp"], c["dst_tp"], c["rank"],
                       CODE[c["src"]], CODE[c["wire"]], ORDER[c["order"]], c["page"], pool, lens,
                       c["src_page"], spool,
                       cache_dtype=CODE[c["cache"]] if c["cache"] != c["wire"] else 0)
    rows = (2 * c["layers"], pool, c["page"], hd)
    st = dict(op=c["op"], paged=c["order"] == "paged", shards=shards, bt=bt, stride=bt.shape[1],
              sbt=sbt, sstride=sbt.shape[1] if sbt is not None else 0, cache=None, scales=None)
    if c["op"] == "noalloc":
        st["desc"] = desc
    else:
        st["plan"] = K.kvx_plan(desc)
    if c["op"] != "pack":
        st["cache"] = torch.zeros((*rows, c["dim"]), device="cuda",
                                  dtype=torch.uint8 if cache8 else TORCH[c["cache"]])
        if cache8:
            st["scales"] = torch.zeros(rows, dtype=torch.float32, device="cuda")
    if c["op"] in ("pack", "pack_unpack"):
        nbytes = K.kvx_plan_info_get(st["plan"]).wire_bytes
        st["wire"] = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
        st["wire_out"] = st["wire"] if c["wire"] in FMAX else st["wire"].view(TORCH[c["wire"]])
    if c["op"] == "pipe":
        st["pipe"] = K.kvx_pipe_create(st["plan"], c["chunk"], c["slots"])
    return st


def run(s):
    op = s["op"]
    if op == "repack":
        if s["paged"]:
            K.kvx_repack_paged(s["plan"], s["shards"], s["sbt"], s["sstride"], s["cache"],
                               s["scales"], s["bt"], s["stride"])
        else:
            K.kvx_repack(s["plan"], s["shards"], s["cache"], s["scales"], s["bt"], s["stride"])
    elif op == "noalloc":
        K.kvx_repack_noalloc(s["desc"], s["shards"], s["cache"], s["scales"], s["bt"], s["stride"])
    elif op == "pipe":
        K.kvx_pipe_run(s["pipe"], s["shards"], s["sbt"], s["sstride"], s["cache"], s["scales"],
                       s["bt"], s["stride"])
    else:
        if s["paged"]:
            K.kvx_pack_paged(s["plan"], s["shards"], s["sbt"], s["sstride"], s["wire"])
        else:
            K.kvx_pack(s["plan"], s["shards"], s["wire"])
        if op == "pack":
            return {"wire": s["wire_out"]}
        K.kvx_unpack(s["plan"], s["wire"], s["cache"], s["scales"], s["bt"], s["stride"])
        return {"wire": s["wire_out"], "cache": s["cache"]} if s["scales"] is None else \
            {"wire": s["wire_out"], "cache": s["cache"], "scales": s["scales"]}
    return {"cache": s["cache"]} if s["scales"] is None else \
        {"cache": s["cache"], "scales": s["scales"]}


def work(case):
    """The rank's rows read once and written once (the transfer tensor as
    well where there is one), their scales, and the block tables."""
    c = case
    lens = lengths(c)
    _, hd = _heads(c)
    rows = 2 * c["layers"] * sum(lens) * hd

    def size(kind):
        return rows * (c["dim"] + 4 if kind in FMAX else 2 * c["dim"])

    nbytes = rows * c["dim"] * 2
    if c["op"] in ("pack", "pack_unpack"):
        nbytes += size(c["wire"]) * (2 if c["op"] == "pack_unpack" else 1)
    if c["op"] != "pack":
        nbytes += size(c["cache"]) + 4 * sum(_pages(lens, c["page"]))
    if c["order"] == "paged":
        nbytes += 4 * sum(_pages(lens, c["src_page"]))
    return {"bytes": nbytes, "flops": 0}


def tolerance(case):
    # copies, correctly rounded casts and codes: one right answer each
    return "exact"


def exact(case, seed):
    """What `run` returns, in 64 bits: values as they are before the cast, row
    scales as the exact quotient.  8-bit codes and transfer tensors that hold
    them are bytes and have no such value."""
    c = case
    lens, shards, bt, pool, sbt, _ = _inputs(c, seed)
    _, hd = _heads(c)
    P, D = 2 * c["layers"], c["dim"]
    cache8, wire8 = c["cache"] in FMAX, c["wire"] in FMAX
    cache = scales = wire = None
    if c["op"] != "pack":
        if cache8:
            scales = torch.zeros((P, pool, c["page"], hd), dtype=torch.float64, device="cuda")
        else:
            cache = torch.zeros((P, pool, c["page"], hd, D), dtype=torch.float64, device="cuda")
    segments, at = [], 0
    for r, T in enumerate(lens):
        n = P * T
        hs, _ = _heads(c)
        t = torch.arange(T, device="cuda")
        heads = []
        for j, h in _rank_heads(c):
            if c["order"] == "paged":
                ids = sbt[r].long()[t // c["src_page"]]
                heads.append(shards[j][:, ids, t % c["src_page"], h])
            else:
                x = shards[j][at * P * hs * D:(at + T) * P * hs * D]
                heads.append(x.view(P, T, hs, D)[:, :, h] if c["order"] == "thd" else
                             x.view(P, hs, T, D)[:, h])
        x = torch.stack(heads, dim=2).double()                  # [plane][token][head][dim]
        at += T
        if c["op"] != "pack":
            ids, slot = bt[r].long()[t // c["page"]], t % c["page"]
            if cache8:
                scales[:, ids, slot] = x.abs().amax(-1) / FMAX[c["cache"]]
            else:
                cache[:, ids, slot] = x
        if c["op"] in ("pack", "pack_unpack") and not wire8:
            flat = x.reshape(-1)
            segments += [flat, flat.new_zeros(-flat.numel() * 2 % 256 // 2)]
    if segments:
        wire = torch.cat(segments)
    if c["op"] == "pack":
        return None if wire8 else {"wire": wire}
    out = {"cache": cache} if not cache8 else {"cache": None, "scales": scales}
    return {"wire": wire, **out} if c["op"] == "pack_unpack" else out
