"""The destination rows' store forms give the same bytes: a cache above 256 MB
is written through the L2, the same cache filled layer by layer (each launch
below that) is not.  Arbitrary 16-bit patterns (NaN and infinities among them)
through copies, casts, codes with scales, and both dequantising forms, whose
lanes store two vectors."""
import pytest
import torch

import paper_2509_17542_amd as K

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

L, H, BS, T = 3, 8, 16, 30011   # one request; 3 layers, 8 heads, a ragged last page


@pytest.mark.parametrize("op", ["repack", "pack_unpack"])
@pytest.mark.parametrize("src,wire,cache,dim", [
    (K.BF16, K.BF16, K.BF16, 128), (K.FP16, K.BF16, K.BF16, 128), (K.BF16, K.E4M3FN, K.E4M3FN, 192),
    (K.BF16, K.E4M3FN, K.BF16, 192), (K.FP16, K.E5M2, K.FP16, 256)])
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
