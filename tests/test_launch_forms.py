"""What the planner's rules choose for a launch, checked on the CPU: the
planner and the launch calls run with the HIP runtime and the kernels replaced
(tests/launch_probe.cpp), so the arguments of every launch can be read."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from cases import random_workloads
from conftest import ROOT
from gpu_util import desc_for
from test_gpu_flat import FLAT as FLAT_CASES
import test_gpu_stores as stores

import paper_2509_17542_amd as K

CSRC = os.path.join(ROOT, "paper_2509_17542_amd", "csrc")
STREAM, THROUGH, CACHED = 0, 1, 2                # kvx_internal.h, Store
ALIGNED, FLAT, FLAT_CACHED = 0, 1, 2             # kvx_internal.h, Form
MODES = ("pack", "unpack", "repack")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or
                                not os.path.exists("/opt/rocm/include/hip"),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("probe") / "probe.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-fPIC", "-shared", "-Wl,-Bsymbolic",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I",
                    "/opt/rocm/include", os.path.join(ROOT, "tests", "launch_probe.cpp"),
                    os.path.join(CSRC, "kvx_plan.cpp"), "-o", so], check=True, capture_output=True)
    lib = ctypes.CDLL(so)
    lib.probe_walk.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32, ctypes.c_int,
                               ctypes.c_void_p]
    lib.kvx_last_error.restype = ctypes.c_char_p
    for name in ("kvx_plan_info_get", "kvx_plan_destroy", "kvx_pack", "kvx_pack_paged", "kvx_unpack",
                 "kvx_repack", "kvx_repack_paged"):
        getattr(lib, name).argtypes = getattr(K._lib, name).argtypes
    return lib


class Launch:
    """One plan in the probe; `launch(mode)` makes the call on made-up aligned
    addresses (nothing reads them) and returns its arguments."""
    BT, STRIDE, SBT = 0x40000, 1 << 22, 0x50000

    def __init__(self, lib, desc):
        self.lib, self.desc, self.plan = lib, desc, ctypes.c_void_p()
        self.ok(lib.kvx_plan(ctypes.byref(desc), ctypes.byref(self.plan)))
        self.info = K.kvx_plan_info()
        self.ok(lib.kvx_plan_info_get(self.plan, ctypes.byref(self.info)))

    def ok(self, status):
        assert status == K.OK, self.lib.kvx_last_error()

    def launch(self, mode):
        d, lib = self.desc, self.lib
        shards = (ctypes.c_void_p * d.src_tp)(*[0x10000] * d.src_tp)
        cache_t = d.cache_dtype or d.dst_dtype
        cache = (0x20000, 0x30000 if cache_t in (K.E4M3FN, K.E5M2) else None, self.BT, self.STRIDE)
        sbt = (self.SBT, self.STRIDE) if d.src_order == K.PAGED else ()
        paged = "_paged" if sbt else ""
        if mode == "pack":
            self.ok(getattr(lib, "kvx_pack" + paged)(self.plan, shards, *sbt, 0x60000, None))
        elif mode == "unpack":
            self.ok(lib.kvx_unpack(self.plan, 0x60000, *cache, None))
        else:
            self.ok(getattr(lib, "kvx_repack" + paged)(self.plan, shards, *sbt, *cache, None))
        v = (ctypes.c_int64 * 8)()
        assert lib.probe_launch(v) == 8
        names = ("form", "store", "units", "planes", "items", "segs", "page_rows", "cpr")
        return dict(zip(names, v))

    def close(self):
        self.lib.kvx_plan_destroy(self.plan)


# A flat launch's lanes follow one another across pages, but what they write
# in one piece ends with the page, whatever the rows of a wave add up to: only
# broken sectors of the shortest pages are left to the L2.
SHORT_PAGES = [(1, 40, 1, K.BF16, CACHED), (1, 48, 1, K.BF16, CACHED), (1, 16, 3, K.BF16, CACHED),
               (1, 80, 1, K.E4M3FN, CACHED), (1, 112, 1, K.E4M3FN, CACHED),
               (1, 16, 5, K.E4M3FN, CACHED), (1, 80, 1, K.BF16, STREAM),
               (1, 112, 1, K.BF16, STREAM), (3, 80, 1, K.BF16, STREAM), (1, 80, 5, K.E4M3FN, STREAM),
               (1, 80, 5, K.BF16, STREAM), (1, 128, 1, K.BF16, STREAM), (2, 96, 1, K.BF16, STREAM)]


@pytest.mark.parametrize("mode", ["unpack", "repack"])
@pytest.mark.parametrize("heads,dim,page,wire,store", SHORT_PAGES)
def test_short_pages(probe, heads, dim, page, wire, store, mode):
    for tokens in (4096, 2_000_000):            # below and above 256 MB of most
        p = Launch(probe, K.make_desc(2, heads, dim, 1, 1, 0, K.BF16, wire, K.THD, page, 1 << 21,
                                      [tokens]))
        a = p.launch(mode)
        p.close()
        assert (a["form"], a["store"]) == (FLAT_CACHED if store == CACHED else FLAT, store)


SMALL, LARGE = 4096, 300_000                    # tokens: 4 layers of 8 x 16 elements or more


@pytest.mark.parametrize("dim,mode,tokens,store", [
    (112, "repack", SMALL, CACHED), (112, "repack", LARGE, CACHED), (112, "unpack", SMALL, STREAM),
    (112, "unpack", LARGE, CACHED), (144, "repack", SMALL, STREAM), (144, "repack", LARGE, STREAM),
    (144, "unpack", SMALL, STREAM), (144, "unpack", LARGE, STREAM), (304, "repack", LARGE, STREAM)])
def test_half_rows(probe, dim, mode, tokens, store):
    """Broken half rows of a dequantising lane: left to the L2 below 128 bytes,
    by the unpack into caches above 256 MB only."""
    p = Launch(probe, K.make_desc(4, 8, dim, 1, 1, 0, K.BF16, K.E4M3FN, K.THD, 16, 1 << 20, [tokens],
                                  cache_dtype=K.BF16))
    assert (tokens * 4 * 2 * 8 * dim * 2 > 256 << 20) == (tokens == LARGE)
    assert p.launch(mode)["store"] == store
    p.close()


@pytest.mark.parametrize("heads,dim,wire,mode,form,store", [
    (2, 112, K.BF16, "pack", ALIGNED, CACHED),      # 224-byte pieces
    (2, 208, K.BF16, "pack", ALIGNED, STREAM),      # 416
    (2, 208, K.BF16, "repack", ALIGNED, CACHED),
    (6, 80, K.BF16, "pack", FLAT_CACHED, CACHED),   # 480, rows packed chunk by chunk
    (2, 464, K.E4M3FN, "pack", ALIGNED, CACHED),    # 464 bytes of codes
    (6, 112, K.BF16, "repack", ALIGNED, STREAM)])   # 672
def test_pieces_of_two_shards(probe, heads, dim, wire, mode, form, store):
    p = Launch(probe, K.make_desc(2, heads, dim, 2, 1, 0, K.BF16, wire, K.THD, 16, 1 << 12, [4096]))
    a = p.launch(mode)
    p.close()
    assert (a["form"], a["store"]) == (form, store)


@pytest.mark.parametrize("mode", ["pack", "repack"])
@pytest.mark.parametrize("dim", [112, 144, 208])
def test_pieces_of_unequal_shards(probe, dim, mode):
    """One head and three of another shard, and the mirror image: the longer
    broken piece decides, in either order."""
    for rank in (1, 3):
        p = Launch(probe, K.make_desc(2, 20, dim, 4, 5, rank, K.BF16, K.BF16, K.THD, 16, 1 << 12,
                                      [4096]))
        a = p.launch(mode)
        p.close()
        assert a["segs"] == 2 and a["store"] == STREAM


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("name", list(FLAT_CASES))
def test_flat_cases_are_flat(probe, name, mode):
    """Every launch of tests/test_gpu_flat.py runs a flat kernel."""
    w = FLAT_CASES[name]
    p = Launch(probe, desc_for(w, w.lens_override))
    a = p.launch(mode)
    p.close()
    assert a["form"] != ALIGNED


@pytest.mark.parametrize("src,wire,cache,dim", stores.TYPES)
def test_store_cases_are_written_through(probe, src, wire, cache, dim):
    """The launches of tests/test_gpu_stores.py: the whole cache is written
    through, one layer of it streamed."""
    for layers, store in ((stores.L, THROUGH), (1, STREAM)):
        p = Launch(probe, K.make_desc(layers, stores.H, dim, 1, 1, 0, src, wire, K.THD, stores.BS,
                                      2000, [stores.T], cache_dtype=0 if cache == wire else cache))
        for mode in ("repack", "unpack"):
            a = p.launch(mode)
            assert (a["form"], a["store"]) == (ALIGNED, store)
        p.close()


RANDOM = {**FLAT_CASES, **random_workloads(31, 160)}


@pytest.mark.parametrize("name", list(RANDOM))
def test_every_row_has_one_lane(probe, name):
    """Page-aligned or flat, each 16-byte chunk of each row of each page is
    taken by exactly one lane, the rows of a quantising launch by aligned
    lanes, and the only request's pages are those of the plan."""
    w = RANDOM[name]
    lens = w.lens_override
    p = Launch(probe, desc_for(w, lens))
    for mode in MODES if p.info.num_items else ():
        a = p.launch(mode)
        assert a["items"] == p.info.num_items
        hits = np.zeros((a["planes"], a["items"], a["segs"], a["page_rows"], a["cpr"]), np.uint8)
        assert probe.probe_walk(p.plan, p.BT if mode != "pack" else None, p.STRIDE,
                                w.dst_dtype in ("e4m3fn", "e5m2"), hits.ctypes.data) == 0
        want = np.zeros_like(hits)
        item = 0
        heads = segments(w) if mode != "unpack" else [w.hd]
        assert len(heads) == a["segs"]
        for t in lens:
            for t0 in range(0, t, w.block_size):
                for sg, n in enumerate(heads):
                    want[:, item, sg, :min(w.block_size, t - t0) * n] = 1
                item += 1
        assert np.array_equal(hits, want), (mode, a)
    p.close()


def segments(w):
    """Heads of each run of the decode rank's heads that lies in one shard."""
    g0 = w.dst_rank * w.hd if w.dst_tp <= w.heads else w.dst_rank // (w.dst_tp // w.heads)
    shard = [(g0 + i) // w.hs for i in range(w.hd)]
    return [shard.count(j) for j in sorted(set(shard))]


def test_random_launches_take_both_forms(probe):
    forms = []
    for name, w in RANDOM.items():
        p = Launch(probe, desc_for(w, w.lens_override))
        if p.info.num_items:
            forms += [(p.launch(m)["form"], w.dst_dtype in ("e4m3fn", "e5m2")) for m in MODES]
        p.close()
    for form in (ALIGNED, FLAT, FLAT_CACHED):
        for codes in (False, True):
            assert forms.count((form, codes)) >= 10, (form, codes)
