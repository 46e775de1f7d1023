"""GPU parity where a launch packs the rows of consecutive pages into its
workgroups (pages that leave page-aligned workgroups partly idle): one-token
pages, one head per rank, chunk counts per row that are not powers of two (up
to one row per wave), head segments of unequal size, pages of many requests
in one workgroup, a last workgroup of one row.  Zero rows, infinities and NaN
among the values, 10% of the page ids outside the pools.  Whole pools and
transfer tensors against the oracle, byte for byte."""
import numpy as np
import pytest
import torch

from cases import FP8, L8B, P8B, QWEN, inputs, oracle_problem, out_of_pool
from gpu_util import gpu_run, log, oracle_pool

import oracle as O
import workload as W

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _w(base, name, lens, **kw):
    nb = sum((t + kw["block_size"] - 1) // kw["block_size"] for t in lens) + 3
    if base is P8B:
        s = kw["src_block_size"]
        kw["src_num_blocks"] = sum((t + s - 1) // s for t in lens) + 2
    return base.replace(name=name, layers=2, total_layers=2, num_requests=len(lens),
                        lens_override=tuple(lens), num_blocks=nb, **kw)


ONES = (1,) * 40
FLAT = {w.name: w for w in [
    _w(QWEN, "token_pages_hd80_tp2to3", (1, 37, 0, 130), src_order="thd", heads=6, head_dim=80,
       src_tp=2, dst_tp=3, dst_rank=1, block_size=1),
    _w(L8B, "one_token_requests", ONES, heads=2, head_dim=64, block_size=8),
    _w(L8B, "unequal_segments", (23, 1, 40), heads=12, head_dim=96, src_tp=3, dst_tp=2,
       block_size=5),
    _w(L8B, "chunks33_bf16", (9, 30), heads=2, head_dim=264, block_size=3),
    _w(FP8, "one_head_e4m3", (70, 3, 129), heads=8, head_dim=128, src_tp=4, dst_tp=8, dst_rank=5,
       block_size=16),
    _w(FP8, "one_lane_rows_e4m3", (1, 65, 200), heads=1, head_dim=16, block_size=1),
    _w(FP8, "rows21_per_wave_e5m2", (40, 22), heads=4, head_dim=48, dst_dtype="e5m2",
       src_order="htd", block_size=3),
    _w(FP8, "one_row_per_wave_e4m3", (17, 6), heads=2, head_dim=528, block_size=1),
    _w(FP8, "chunks62_e4m3_bf16", (11, 4), heads=1, head_dim=992, cache_dtype="bf16",
       block_size=2),
    _w(P8B, "paged3_hd112_e5m2_bf16", (50, 0, 7), heads=4, head_dim=112, dst_dtype="e5m2",
       cache_dtype="bf16", dst_tp=2, block_size=5, src_block_size=3),
    _w(P8B, "paged_one_head_bf16_fp16", (33, 90), heads=4, head_dim=64, dst_dtype="fp16",
       dst_tp=8, dst_rank=3, block_size=16, src_block_size=16),
]}


def _case(name):
    w = FLAT[name]
    lens, bt, stride, shards = inputs(w)
    rng = np.random.default_rng(5)
    inf = 0x7C00 if w.src_dtype == "fp16" else 0x7F80
    for s in shards:
        if s is not None:
            rows = s.reshape(-1, w.head_dim)
            pick = rng.permutation(len(rows))[:max(4, len(rows) // 8)]
            for k, v in enumerate((0, 0x8000, inf, 0x7FFF, 0xFFFF)):  # +-0 rows, infinity, NaN
                rows[pick[k::5], :w.head_dim if k < 2 else 1 + k] = v
    sbt = None
    if w.src_order == "paged":
        sbt = out_of_pool(W.src_block_table(w, lens)[0], w.src_num_blocks, rng)
    return w, lens, out_of_pool(bt, w.num_blocks, rng), stride, shards, sbt


def _eq(a, b):
    return np.array_equal(np.asarray(a).view(np.uint8), np.asarray(b).view(np.uint8))


@pytest.mark.parametrize("name", list(FLAT))
def test_flat(name):
    w, lens, bt, stride, shards, sbt = _case(name)
    log(f"flat {name}: H={w.heads} D={w.head_dim} bs={w.block_size} lens={list(lens)}")
    cache, scales, _ = gpu_run("repack", w, lens, bt, stride, shards, sbt=sbt)
    want_c, want_s = oracle_pool(w, lens, bt, stride, shards, sbt=sbt)
    assert _eq(cache.cpu().numpy(), want_c)
    if want_s is not None:
        assert _eq(scales.cpu().numpy(), want_s)
    _, _, wire = gpu_run("pack", w, lens, bt, stride, shards, sbt=sbt)
    want = O.pack(oracle_problem(O, w, lens, sbt=sbt), shards)
    assert _eq(wire.cpu().numpy()[:want.size], want)
    cache, scales, _ = gpu_run("unpack", w, lens, bt, stride, None, wire_in=want, sbt=sbt)
    want_c, want_s = oracle_pool(w, lens, bt, stride, shards, op="unpack", wire=want, sbt=sbt)
    assert _eq(cache.cpu().numpy(), want_c)
    if want_s is not None:
        assert _eq(scales.cpu().numpy(), want_s)
