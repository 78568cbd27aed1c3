"""Generic projection: the small product, which rotates its results itself, gives a row the bits of the large one with its rotation
in a second kernel (the sums run in the same order, the angles are taken alike)."""
import ctypes as C

import pytest
import torch

from paper_2604_08585_amd import binding as qb
from paper_2604_08585_amd import inputs
from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,K,H,Hkv,D,style", [
    ("f32", 256, 4, 2, 64, 0), ("f32", 72, 3, 1, 128, 1), ("f32", 256, 4, 2, 64, 1), ("bf16", 72, 6, 3, 64, 0)])
def test_small_product_rotates_as_the_large_one(dtype, K, H, Hkv, D, style):
    print(f"generic projection {dtype} K={K} H={H}/{Hkv} D={D} style={style}", flush=True)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    sh = inputs.LayerShape(K, H, Hkv, D, 10000.0, dtype, style)
    desc = qb.make_desc(sh)
    M = 64 * (256 * 64 // sh.qkv_rows + 2)               # from 256 large tiles on
    g = torch.Generator(device=DEV).manual_seed(K + D)
    x, w = (torch.randn(s, generator=g, device=DEV, dtype=dt) for s in ((M, K), (sh.qkv_rows, K)))
    pos = torch.randint(-3, 1 << 26, (M,), generator=g, device=DEV).int()
    gather = torch.randperm(M, generator=g, device=DEV).int()
    gather[5] = M                                        # outside x: a zero row
    dst = torch.randperm(M, generator=g, device=DEV).int()
    dst[3], dst[7] = -1, M                               # not in the cache

    def run(m, q=True):
        out = [torch.full((m, h, D), 7.0, dtype=dt, device=DEV) for h in (H, Hkv, Hkv)]
        cache = [torch.full((M, Hkv, D), 7.0, dtype=dt, device=DEV) for _ in range(2)]
        qb.qcf_recompute_qkv_scatter(desc, x, M, gather, m, w, pos, out[0] if q else None, out[1], out[2], dst, *cache, M)
        torch.cuda.synchronize()
        return out + cache

    whole = run(M)
    for m in (1, 16, 77):
        part = run(m, q=m != 16)
        for i, (a, b) in enumerate(zip(part[:3], whole)):
            assert bool((a == 7.0).all()) if i == 0 and m == 16 else torch.equal(a, b[:m])
        rows = dst[:m].long()
        rows = rows[(rows >= 0) & (rows < M)]
        for a, b in zip(part[3:], whole[3:]):
            want = torch.full_like(b, 7.0)
            want[rows] = b[rows]
            assert torch.equal(a, want)
