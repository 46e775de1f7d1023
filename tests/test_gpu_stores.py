"""The destination rows' store forms give the same bytes: a cache above 256 MB
is written through the L2, the same cache filled layer by layer (each launch
below that) is not.  Arbitrary 16-bit patterns (NaN and infinities among them)
through copies, casts, codes with scales, and both dequantising forms, whose
lanes store two vectors.  One plane of the written-through cache against the
oracle, byte for byte."""
import numpy as np
import pytest
import torch

import oracle as O

import paper_2509_17542_amd as K

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

ORC = {K.BF16: O.BF16, K.FP16: O.FP16, K.E4M3FN: O.E4M3FN, K.E5M2: O.E5M2}
L, H, BS, T = 3, 8, 16, 30011   # one request; 3 layers, 8 heads, a ragged last page
TYPES = [(K.BF16, K.BF16, K.BF16, 128), (K.FP16, K.BF16, K.BF16, 128),
         (K.BF16, K.E4M3FN, K.E4M3FN, 192), (K.BF16, K.E4M3FN, K.BF16, 192),
         (K.FP16, K.E5M2, K.FP16, 256)]


@pytest.mark.parametrize("op", ["repack", "pack_unpack"])
@pytest.mark.parametrize("src,wire,cache,dim", TYPES)
def test_store_forms(src, wire, cache, dim, op):
    print(f"stores {op} {src}->{wire}->{cache} dim {dim}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(7)
    nb = (T + BS - 1) // BS + 5
    x = torch.randint(-32768, 32768, (L * 2 * T * H * dim,), generator=g, device="cuda",
                      dtype=torch.int16)
    bt = torch.randperm(nb, generator=torch.Generator().manual_seed(1))[:(T + BS - 1) // BS]
    bt = bt.to(torch.int32).reshape(1, -1).cuda()
    esz = 1 if cache in (K.E4M3FN, K.E5M2) else 2
    row = dim * esz
    assert L * 2 * T * H * row > 256 << 20 and 2 * nb * BS * H * row < 256 << 20
    got = []
    for ranges in ([(0, L)], [(l, 1) for l in range(L)]):
        pool = torch.full((L * 2 * nb * BS * H * row,), 0xA5, dtype=torch.uint8, device="cuda")
        scales = torch.zeros(L * 2 * nb * BS * H, device="cuda") if esz == 1 else None
        for l0, n in ranges:
            plan = K.kvx_plan(K.make_desc(n, H, dim, 1, 1, 0, src, wire, K.THD, BS, nb, [T], 0, 0, l0,
                                          L, l0, L, cache_dtype=0 if cache == wire else cache))
            if op == "repack":
                K.kvx_repack(plan, [x], pool, scales, bt, bt.shape[1])
            else:
                w = torch.empty(K.kvx_plan_info_get(plan).wire_bytes, dtype=torch.uint8,
                                device="cuda")
                K.kvx_pack(plan, [x], w)
                K.kvx_unpack(plan, w, pool, scales, bt, bt.shape[1])
        torch.cuda.synchronize()
        got.append((pool, scales))
    assert torch.equal(got[0][0], got[1][0])
    if esz == 1:
        assert torch.equal(got[0][1].view(torch.int32), got[1][1].view(torch.int32))
    # layer 1's values against a one-layer problem of the oracle
    p = O.OracleProblem(1, H, dim, 1, 1, 0, ORC[src], ORC[wire], O.TOKEN_MAJOR, BS, nb, [T],
                        cache_fmt=0 if cache == wire else ORC[cache])
    n = 2 * T * H * dim
    want, want_s = O.expected_rows(p, [x[n:2 * n].cpu().numpy().view(np.uint16)], 0, 0, 1, 0, T)
    ids = bt[0].long()
    plane = got[0][0].view(2 * L, nb, BS * H * row)[3, ids].cpu().numpy().reshape(-1, row)
    assert np.array_equal(plane[:T * H], want)
    assert (plane[T * H:] == 0xA5).all()
    if esz == 1:
        plane = got[0][1].view(2 * L, nb, BS * H)[3, ids].cpu().numpy().reshape(-1)
        assert np.array_equal(plane[:T * H].view(np.uint32), want_s.view(np.uint32))
