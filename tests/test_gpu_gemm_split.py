"""Products whose contraction is split, against float32: over 256 x 256 tiles (ragged rows, an odd number of column blocks,
ranges of unequal length, the rotation and the gated SiLU behind the reduction), and weight streams for few rows."""
import ctypes as C

import pytest
import torch

import host_rules
from paper_2604_08585_amd import binding as qb
from paper_2604_08585_amd import inputs
from gpu_util import DEV

pytestmark = pytest.mark.gpu
BF = torch.bfloat16
DESC = inputs.LayerShape(4096, 32, 8, 128, 500000.0, "bf16")


def _normal(seed, *size, std=1.0):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return (torch.randn(size, generator=g, device=DEV) * std).to(BF)


def _one_rounding(got, ref, slack=2e-4):
    err = (got.float() - ref).abs()
    assert bool((err <= 2.0 ** -8 * ref.abs() + slack).all()), float(err.max())


def _sums(M, N, splits):
    """Workspace of a contraction in `splits` ranges over 256 x 256 tiles."""
    return splits * ((M + 255) // 256 * 256) * N * 4


@pytest.mark.parametrize("M,K,N,splits,res", [
    (1229, 14336, 4096, 3, True),        # 76, 76 and 72 k-tiles; 205 rows in the last row tile
    (765, 14336, 3456, 6, True),         # an odd number of column blocks, a last range of 34
    (1025, 14336, 3712, 3, False),       # one row in the last row tile
    (129, 14336, 8448, 6, False),        # one row tile
    (512, 8192, 10240, 3, True)])
def test_linear(M, K, N, splits, res):
    print(f"split product M={M} K={K} N={N}", flush=True)
    desc = qb.make_desc(DESC)
    assert qb.qcf_linear_workspace_bytes(desc, M, K, N) == _sums(M, N, splits)
    x, w = _normal(1, M, K), _normal(2, N, K, std=K ** -0.5)
    r = _normal(3, M, N) if res else None
    ref = x.float() @ w.float().T + (r.float() if res else 0.0)
    outs = []
    for _ in range(2):
        out = torch.full((M + 1, N), 7.0, dtype=BF, device=DEV)
        qb.qcf_linear(desc, x, M, K, w, N, r, out)
        outs.append(out)
    torch.cuda.synchronize()
    _one_rounding(outs[0][:M], ref)
    assert torch.equal(outs[0], outs[1]) and bool((outs[0][M] == 7.0).all())


@pytest.mark.parametrize("M,K,N,splits", [
    (1, 14336, 4096, 8), (61, 14336, 4096, 8), (64, 8192, 8192, 3),      # 43, 43 and 42 k-tiles
    (65, 4096, 6144, 4), (110, 8192, 8192, 3), (128, 14336, 2048, 14)])
def test_weight_stream(M, K, N, splits):
    """One row tile of 64 or 128 rows: the ranges that its weight stream is cut into."""
    print(f"weight stream M={M} K={K} N={N}", flush=True)
    desc = qb.make_desc(DESC)
    assert qb.qcf_linear_workspace_bytes(desc, M, K, N) == splits * (64 if M <= 64 else 128) * N * 4
    x, w, r = _normal(9, M, K), _normal(10, N, K, std=K ** -0.5), _normal(11, M, N)
    out = torch.full((M + 1, N), 7.0, dtype=BF, device=DEV)
    qb.qcf_linear(desc, x, M, K, w, N, r, out)
    torch.cuda.synchronize()
    _one_rounding(out[:M], x.float() @ w.float().T + r.float())
    assert bool((out[M] == 7.0).all())


def test_projection_with_write_back():
    M, dm, H, Hkv, D = 400, 8192, 64, 8, 128
    print(f"split projection M={M} H={H}", flush=True)
    sh = inputs.LayerShape(dm, H, Hkv, D, 500000.0, "bf16")
    desc = qb.make_desc(sh)
    assert qb.qcf_recompute_qkv_workspace_bytes(desc, M) == _sums(M, sh.qkv_rows, 3)
    x, w = _normal(4, M + 50, dm), _normal(5, sh.qkv_rows, dm, std=dm ** -0.5)
    g = torch.Generator(device=DEV).manual_seed(6)
    gather = torch.randperm(M + 50, generator=g, device=DEV)[:M].int()
    gather[17] = -1                                          # outside x: a zero row
    pos = torch.randint(0, 40000, (M,), generator=g, device=DEV).int()
    dst = torch.randperm(M + 50, generator=g, device=DEV)[:M].int()
    q, k, v = (torch.full((M, h, D), 7.0, dtype=BF, device=DEV) for h in (H, Hkv, Hkv))
    kf, vf = (torch.full((M + 50, Hkv, D), 7.0, dtype=BF, device=DEV) for _ in range(2))
    qb.qcf_recompute_qkv_scatter(desc, x, M + 50, gather, M, w, pos, q, k, v, dst, kf, vf, M + 50)
    torch.cuda.synchronize()
    xs = x[gather.clamp(min=0).long()].float()
    xs[17] = 0
    y = (xs @ w.float().T).reshape(M, H + 2 * Hkv, D)
    theta = 500000.0 ** (-torch.arange(0, D, 2, device=DEV, dtype=torch.float64) / D)
    ang = pos.double()[:, None, None] * theta
    a, b = y[:, :H + Hkv, :D // 2].double(), y[:, :H + Hkv, D // 2:].double()
    y[:, :H + Hkv] = torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1).float()
    for got, ref in ((q, y[:, :H]), (k, y[:, H:H + Hkv]), (v, y[:, H + Hkv:])):
        _one_rounding(got, ref)
    for fused, new in ((kf, k), (vf, v)):
        ref = torch.full_like(fused, 7.0)
        ref[dst.long()] = new
        assert torch.equal(fused, ref)


def test_gated_silu():
    """Gate and up are rounded to bf16 before the activation: |error| <= 3 roundings of the product of their sizes."""
    M, K, F = 512, 8192, 5120
    print(f"split gated product M={M} F={F}", flush=True)
    desc = qb.make_desc(DESC)
    assert qb.load_library().qcf_linear_swiglu_workspace_bytes(C.byref(desc), M, K, F) == _sums(M, 2 * F, 3)
    x, w = _normal(7, M, K), _normal(8, 2 * F, K, std=K ** -0.5)
    out = torch.full((M, F), 7.0, dtype=BF, device=DEV)
    qb.qcf_linear_swiglu(desc, x, M, K, w, F, out)
    torch.cuda.synchronize()
    y = (x.float() @ w.float().T).to(BF).float()             # (a sum near a rounding boundary may round the other way)
    gate, up = y[:, :F], y[:, F:]
    ref = torch.nn.functional.silu(gate) * up
    err = (out.float() - ref).abs()
    assert bool((err <= 2.0 ** -8 * ref.abs() + 2.0 ** -7 * (1.1 * gate.abs() * up.abs()) + 2e-4).all()), float(err.max())


@pytest.mark.parametrize("M,K,F", [
    (16, 1024, 2816), (200, 1024, 2816),     # 44 column blocks over 16 k-tiles; one and two row tiles
    (1, 64, 16448), (40, 128, 14336),        # one and two k-tiles, fewer than the loads on their way
    (61, 4096, 14336), (128, 2048, 8192)])
def test_gated_weight_stream(M, K, F):
    """Few rows, undivided.  Bounds as above."""
    print(f"gated weight stream M={M} K={K} F={F}", flush=True)
    desc = qb.make_desc(DESC)
    assert qb.load_library().qcf_linear_swiglu_workspace_bytes(C.byref(desc), M, K, F) == 0
    x, w = _normal(12, M, K), _normal(13, 2 * F, K, std=K ** -0.5)
    outs = []
    for _ in range(2):
        out = torch.full((M + 1, F), 7.0, dtype=BF, device=DEV)
        qb.qcf_linear_swiglu(desc, x, M, K, w, F, out)
        outs.append(out)
    torch.cuda.synchronize()
    y = (x.float() @ w.float().T).to(BF).float()
    gate, up = y[:, :F], y[:, F:]
    ref = torch.nn.functional.silu(gate) * up
    err = (outs[0][:M].float() - ref).abs()
    assert bool((err <= 2.0 ** -8 * ref.abs() + 2.0 ** -7 * (1.1 * gate.abs() * up.abs()) + 2e-4).all()), float(err.max())
    assert torch.equal(outs[0], outs[1]) and bool((outs[0][M] == 7.0).all())


@pytest.mark.parametrize("M,K,F", [(513, 4096, 14336), (600, 2048, 8192), (700, 1024, 2816)])
def test_gated_product_without_workspace_has_one_order_of_sums(M, K, F):
    """Without a workspace a row's bits depend neither on the number of rows nor on its place among them: whole rounds of 256 x 256
    tiles and a remainder of one row (the first shape), other tiles than those of a batch cut short."""
    print(f"order of sums of the gated product M={M} K={K} F={F}", flush=True)
    desc, lib = qb.make_desc(DESC), qb.load_library()
    x, w = _normal(14, M, K), _normal(15, 2 * F, K, std=K ** -0.5)
    x[M - 1] = x[3]

    def product(rows):
        out = torch.full((rows, F), 7.0, dtype=BF, device=DEV)
        st = torch.cuda.current_stream().cuda_stream
        assert lib.qcf_linear_swiglu(C.byref(desc), x.data_ptr(), rows, K, w.data_ptr(), F, out.data_ptr(), None, 0, st) == 0
        torch.cuda.synchronize()
        return out

    whole = product(M)
    assert torch.equal(whole[M - 1], whole[3])
    for rows in (4, 61, 128):
        assert torch.equal(product(rows), whole[:rows]), rows


@pytest.mark.parametrize("M,D,style,far", [(33, 64, 0, False), (1, 64, 1, True), (70, 128, 1, False), (128, 128, 0, True)])
def test_rotation_behind_the_reduction(M, D, style, far):
    """The reduction finishes 64 columns of a block in a workgroup: every layout of rotary pairs, zero rows, rows past the last."""
    dm, H, Hkv = 4096, 16, 4
    print(f"reduction M={M} D={D} style={style} far={far}", flush=True)
    sh = inputs.LayerShape(dm, H, Hkv, D, 500000.0, "bf16", style)
    desc = qb.make_desc(sh)
    assert qb.qcf_recompute_qkv_workspace_bytes(desc, M) > 0           # (the contraction is split)
    x, w = _normal(15, M + 5, dm), _normal(16, sh.qkv_rows, dm, std=dm ** -0.5)
    g = torch.Generator(device=DEV).manual_seed(17)
    gather = torch.randperm(M + 5, generator=g, device=DEV)[:M].int()
    gather[M // 2] = M + 5                                   # outside x: a zero row
    pos = torch.randint(0, 2 ** 31 - 1 if far else 40000, (M,), generator=g, device=DEV).int()
    dst = torch.randperm(M + 5, generator=g, device=DEV)[:M].int()
    q, k, v = (torch.full((M + 1, h, D), 7.0, dtype=BF, device=DEV) for h in (H, Hkv, Hkv))
    kf, vf = (torch.full((M + 5, Hkv, D), 7.0, dtype=BF, device=DEV) for _ in range(2))
    qb.qcf_recompute_qkv_scatter(desc, x, M + 5, gather, M, w, pos, q, k, v, dst, kf, vf, M + 5)
    torch.cuda.synchronize()
    xs = x[gather.clamp(max=M + 4).long()].float()
    xs[M // 2] = 0
    y = (xs @ w.float().T).reshape(M, H + 2 * Hkv, D).double()
    ang = pos.double()[:, None, None] * 500000.0 ** (-torch.arange(0, D, 2, device=DEV, dtype=torch.float64) / D)
    even, odd = (slice(0, D // 2), slice(D // 2, D)) if style == 0 else (slice(0, D, 2), slice(1, D, 2))
    a, b = y[:, :H + Hkv, even].clone(), y[:, :H + Hkv, odd].clone()
    y[:, :H + Hkv, even] = a * ang.cos() - b * ang.sin()
    y[:, :H + Hkv, odd] = b * ang.cos() + a * ang.sin()
    for got, ref in ((q, y[:, :H]), (k, y[:, H:H + Hkv]), (v, y[:, H + Hkv:])):
        _one_rounding(got[:M], ref.float())
        assert bool((got[M] == 7.0).all())
    for fused, new in ((kf, k), (vf, v)):
        ref = torch.full_like(fused, 7.0)
        ref[dst.long()] = new[:M]
        assert torch.equal(fused, ref)


@pytest.mark.parametrize("M,K,height", [
    (65, 4096, 64), (320, 4096, 64), (321, 4096, 96), (480, 4096, 96), (481, 4096, 128), (641, 4096, 160), (800, 4096, 160),
    (801, 4096, 192), (960, 4096, 192), (961, 4096, 224), (1120, 4096, 224), (1121, 4096, 256), (300, 64, 96), (700, 8192, 160)])
def test_tiles_of_every_height(M, K, height):
    """Launches that fit one round in tiles of 64 to 256 rows: a whole last tile and one of a single row, fewer k-tiles than stages; a
    row's bits are those of a launch of few rows."""
    dm, H, Hkv, D = K, 32, 8, 128
    print(f"tiles of {height} rows M={M} K={K}", flush=True)
    sh = inputs.LayerShape(dm, H, Hkv, D, 500000.0, "bf16")
    desc, lib = qb.make_desc(sh), qb.load_library()
    assert host_rules.tile_rows(M, sh.qkv_rows, K) == height
    x, w = _normal(20, M, dm), _normal(21, sh.qkv_rows, dm, std=dm ** -0.5)
    g = torch.Generator(device=DEV).manual_seed(22)
    gather = torch.randperm(M, generator=g, device=DEV).int()
    gather[M // 3] = -1                                      # outside x: a zero row
    pos = torch.randint(0, 40000, (M,), generator=g, device=DEV).int()
    dst = torch.randperm(M, generator=g, device=DEV).int()

    def project(first, rows):
        q, k, v = (torch.full((rows + 1, h, D), 7.0, dtype=BF, device=DEV) for h in (H, Hkv, Hkv))
        kf, vf = (torch.full((M, Hkv, D), 7.0, dtype=BF, device=DEV) for _ in range(2))
        part = [t[first:first + rows].contiguous() for t in (gather, pos, dst)]
        st = torch.cuda.current_stream().cuda_stream
        assert lib.qcf_recompute_qkv_scatter(C.byref(desc), x.data_ptr(), M, part[0].data_ptr(), rows, w.data_ptr(), part[1].data_ptr(),
                                             q.data_ptr(), k.data_ptr(), v.data_ptr(), part[2].data_ptr(), kf.data_ptr(), vf.data_ptr(),
                                             M, None, 0, st) == 0
        torch.cuda.synchronize()
        assert all(bool((t[rows] == 7.0).all()) for t in (q, k, v))
        assert torch.equal(kf[part[2].long()], k[:rows]) and torch.equal(vf[part[2].long()], v[:rows])
        return [t[:rows] for t in (q, k, v)]

    whole = project(0, M)
    for first in (0, M - min(M, 64)):
        rows = min(M, 64)
        assert host_rules.tile_rows(rows, sh.qkv_rows, K) in (64, 128)
        for a, b in zip(whole, project(first, rows)):
            assert torch.equal(a[first:first + rows], b)
    y = x[gather.clamp(min=0).long()].float() @ w.float().T
    y[M // 3] = 0
    _one_rounding(whole[2].flatten(1), y[:, (H + Hkv) * D:])
