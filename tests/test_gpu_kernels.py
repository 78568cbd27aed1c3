"""GPU parity of the kernel variants that sizes, types and alignment choose between, at the sizes where each can go
wrong (edges of tiles, remainders, smallest and largest of a range), against plain float32 PyTorch or the CPU oracle."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import qcf_oracle as orc
from paper_2604_08585_amd import binding as qb
from paper_2604_08585_amd import inputs, pipeline
from gpu_util import DEV, i32, i64, to_np

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


def say(msg):
    print(msg, flush=True)


def gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def one_rounding(got, ref):
    """One rounding to bf16 of a float32 sum (bound per element)."""
    err = (got.float() - ref).abs()
    assert bool((err <= 2.0 ** -8 * ref.abs() + 2e-4).all()), float(err.max())


@pytest.mark.parametrize("M,K,N,res", [
    (5000, 2048, 8320, True),        # 256 x 256 tiles: ragged rows, an odd number of column blocks
    (2600, 4096, 6144, False),       # 256 x 256 tiles for the full rounds, smaller tiles for the rest
    (61, 2048, 1024, True), (64, 4096, 4096, False), (65, 4096, 1024, True), (128, 4096, 6144, False),   # split contraction
    (1, 1088, 384, True)])           # 17 k-tiles: ranges of unequal length
def test_linear_tile_choices(M, K, N, res):
    """Every tile shape of the bf16 product, with and without the optional workspace, against float32."""
    say(f"linear tiles M={M} K={K} N={N}")
    g = gen(44)
    x = torch.randn((M, K), generator=g, device=DEV, dtype=BF)
    w = torch.randn((N, K), generator=g, device=DEV, dtype=BF) * K ** -0.5
    r = torch.randn((M, N), generator=g, device=DEV, dtype=BF) if res else None
    desc = qb.make_desc(inputs.LayerShape(4096, 32, 8, 128, 500000.0, "bf16"))
    out = torch.full((M, N), 7.0, dtype=BF, device=DEV)
    qb.qcf_linear(desc, x, M, K, w, N, r, out)
    plain = torch.full((M, N), 7.0, dtype=BF, device=DEV)
    assert qb.load_library().qcf_linear(C.byref(desc), x.data_ptr(), M, K, w.data_ptr(), N, r.data_ptr() if res else None,
                                        plain.data_ptr(), None, 0, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    ref = x.float() @ w.float().T + (r.float() if res else 0.0)
    one_rounding(out, ref)
    one_rounding(plain, ref)


def _rotate(y, pos, base, style):
    """Rotary embedding of y [M, heads, d] in float64 angles."""
    d = y.shape[-1]
    theta = base ** (-2.0 * torch.arange(d // 2, device=y.device, dtype=torch.float64) / d)
    ang = pos.double()[:, None] * theta
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = (y[..., :d // 2], y[..., d // 2:]) if style == 0 else (y[..., 0::2], y[..., 1::2])
    a, b = a.double(), b.double()
    ra, rb = a * c - b * s, b * c + a * s
    return torch.cat([ra, rb], -1).float() if style == 0 else torch.stack([ra, rb], -1).flatten(-2).float()


@pytest.mark.parametrize("M,dm,H,Hkv,D,style", [
    (4700, 2048, 32, 8, 128, 0), (4700, 2048, 32, 8, 128, 1), (4700, 2048, 64, 16, 64, 0),   # 256 x 256 tiles
    (60, 2048, 8, 2, 128, 0), (60, 2048, 8, 2, 64, 1), (127, 2048, 8, 2, 64, 0)])             # split contraction
def test_projection_tile_choices(M, dm, H, Hkv, D, style):
    """Rotation, gathering (indices outside x give zero rows), and the write-back, for positions up to 2^31."""
    say(f"projection tiles M={M} H={H} Hkv={Hkv} D={D} style={style}")
    sh = inputs.LayerShape(dm, H, Hkv, D, 500000.0, "bf16", style)
    g = gen(45)
    rows = M + 50
    x = torch.randn((rows, dm), generator=g, device=DEV, dtype=BF)
    w = torch.randn((sh.qkv_rows, dm), generator=g, device=DEV, dtype=BF) * dm ** -0.5
    gather = torch.randperm(rows, generator=g, device=DEV)[:M].int()
    gather[M // 2] = -1
    pos = torch.randint(0, 40000, (M,), generator=g, device=DEV).int()
    pos[:3] = torch.tensor([(1 << 24) + 7, 2 ** 31 - 1, -5], dtype=torch.int32)
    dst = torch.randperm(rows, generator=g, device=DEV)[:M].int()
    dst[1] = rows
    q, k, v = (torch.full((M, h, D), 7.0, dtype=BF, device=DEV) for h in (H, Hkv, Hkv))
    kf, vf = (torch.full((rows, Hkv, D), 7.0, dtype=BF, device=DEV) for _ in range(2))
    qb.qcf_recompute_qkv_scatter(qb.make_desc(sh), x, rows, gather, M, w, pos, q, k, v, dst, kf, vf, rows)
    torch.cuda.synchronize()
    xs = x[gather.clamp(min=0).long()].float()
    xs[M // 2] = 0
    y = (xs @ w.float().T).reshape(M, H + 2 * Hkv, D)
    y[:, :H + Hkv] = _rotate(y[:, :H + Hkv], pos, 500000.0, style)
    for got, ref in ((q, y[:, :H]), (k, y[:, H:H + Hkv]), (v, y[:, H + Hkv:])):
        one_rounding(got, ref)
    keep = torch.ones(M, dtype=torch.bool, device=DEV)
    keep[1] = False
    for fused, new in ((kf, k), (vf, v)):
        ref = torch.full_like(fused, 7.0)
        ref[dst[keep].long()] = new[keep]
        assert torch.equal(fused, ref)
