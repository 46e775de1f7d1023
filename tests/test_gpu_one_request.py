"""GPU parity of launches whose pages all belong to one request (no work-item
table): alone, and between empty requests, whose block-table rows are skipped;
every source order, 16-bit and 8-bit transfer tensors, repack, pack, unpack
and the allocation-free repack.  Whole pools and transfer tensors against the
oracle, byte for byte."""
import numpy as np
import pytest
import torch

from cases import FP8, L8B, P8B, QWEN, inputs, oracle_problem, out_of_pool
from gpu_util import DEV, desc_for, dev_u16, gpu_run, log, oracle_pool, pool

import oracle as O
import workload as W

import paper_2509_17542_amd as K

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

BASES = {"thd_bf16": (L8B, {}), "htd_fp16_bf16": (QWEN, {}), "thd_e4m3_tp1to8": (FP8, dict(dst_tp=8)),
         "paged_bf16": (P8B, dict(src_num_blocks=24)),
         "thd_e5m2_fp16": (FP8, dict(dst_dtype="e5m2", cache_dtype="fp16"))}


def _eq(a, b):
    return np.array_equal(np.asarray(a).view(np.uint8), np.asarray(b).view(np.uint8))


@pytest.mark.parametrize("lens", [(1,), (70,), (0, 0, 131), (0, 37, 0, 0)], ids=str)
@pytest.mark.parametrize("name", list(BASES))
def test_one_request(name, lens):
    base, kw = BASES[name]
    w = base.replace(name=name, layers=2, total_layers=2, num_requests=len(lens),
                     lens_override=lens, block_size=16, num_blocks=12, **kw)
    lens, bt, stride, shards = inputs(w)
    log(f"one request {name} lens={list(lens)}")
    sbt = W.src_block_table(w, lens)[0] if w.src_order == "paged" else None
    rng = np.random.default_rng(3)
    bt = out_of_pool(bt, w.num_blocks, rng)
    want_c, want_s = oracle_pool(w, lens, bt, stride, shards, sbt=sbt)

    def check(cache, scales, what):
        assert _eq(cache.cpu().numpy(), want_c), what
        if want_s is not None:
            assert _eq(scales.cpu().numpy(), want_s), what

    check(*gpu_run("repack", w, lens, bt, stride, shards, sbt=sbt)[:2], "repack")
    cache, scales, wire = gpu_run("pack_unpack", w, lens, bt, stride, shards, sbt=sbt)
    want = O.pack(oracle_problem(O, w, lens, sbt=sbt), shards)
    assert _eq(wire.cpu().numpy()[:want.size], want)
    check(cache, scales, "pack and unpack")
    if w.src_order != "paged":
        cache, scales = pool(w, w.layers)
        dsh = [dev_u16(s) for s in shards]
        bt_d = torch.from_numpy(bt).to(DEV)
        K.kvx_repack_noalloc(desc_for(w, lens), dsh, cache, scales, bt_d, stride)
        torch.cuda.synchronize()
        check(cache, scales, "allocation-free repack")
