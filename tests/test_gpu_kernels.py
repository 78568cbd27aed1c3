"""GPU parity of the kernel variants that sizes, types and alignment choose between, at the sizes where each can go
wrong (edges of tiles, remainders, smallest and largest of a range), against plain float32 PyTorch or the CPU oracle."""
import ctypes as C
import math

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
    (2458, 14336, 4096, True), (2300, 4160, 4096, True), (4916, 4096, 10240, False),   # whole rounds of row tiles, then the rows left
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


@pytest.mark.parametrize("M,K,F", [
    (1300, 2048, 8256),              # 256 x 256 tiles, an odd number of 128-column blocks
    (2600, 4096, 3072),              # 256 x 256 tiles for the full rounds, smaller tiles for the rest
    (4916, 4096, 5120),              # whole rounds of row tiles, then the rows left
    (1, 1088, 64), (61, 4096, 1408), (100, 2048, 512),         # one block; split contraction with 64- and 128-row tiles
    (130, 64, 192),                  # a single k-tile
    (33, 72, 128), (33, 128, 72)])   # K or F that the tiles do not cover: through the workspace
def test_linear_swiglu(M, K, F):
    """The activation in the product's epilogue gives what the two separate calls give (the sums of an element run in
    the same order and gate and up are rounded to bf16 first: bit for bit), with and without the optional workspace."""
    say(f"linear + swiglu M={M} K={K} F={F}")
    g = gen(46)
    x = torch.randn((M, K), generator=g, device=DEV, dtype=BF)
    w = torch.randn((2 * F, K), generator=g, device=DEV, dtype=BF) * (3.0 * K ** -0.5)
    desc = qb.make_desc(inputs.LayerShape(4096, 32, 8, 128, 500000.0, "bf16"))
    gu = torch.empty((M, 2 * F), dtype=BF, device=DEV)
    want = torch.empty((M, F), dtype=BF, device=DEV)
    out = torch.full((M, F), 7.0, dtype=BF, device=DEV)
    qb.qcf_linear(desc, x, M, K, w, 2 * F, None, gu)
    qb.qcf_swiglu(desc, gu, M, F, want)
    qb.qcf_linear_swiglu(desc, x, M, K, w, F, out)
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    lib = qb.load_library()
    plain = torch.full((M, F), 7.0, dtype=BF, device=DEV)
    rc = lib.qcf_linear_swiglu(C.byref(desc), x.data_ptr(), M, K, w.data_ptr(), F, plain.data_ptr(), None, 0,
                               torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    if K % 64 or F % 64:
        assert rc == 3                # QCF_ERR_WORKSPACE_TOO_SMALL
    else:
        assert rc == 0
        # one contraction instead of several ranges: gate and up may round to the neighbouring bf16 value, and
        # silu's slope is at most 1.1
        lim = 2.0 ** -7 * (1.1 * gu[:, :F].float().abs() * gu[:, F:].float().abs() + want.float().abs()) + 2.0 ** -8 * want.float().abs() + 1e-3
        assert bool(((plain.float() - want.float()).abs() <= lim).all())


def test_linear_of_more_column_blocks_than_a_grid_dimension_holds():
    say("linear N=2^23")
    M, K, N = 3, 64, 128 * 65536
    g = gen(57)
    x = torch.randn((M, K), generator=g, device=DEV, dtype=BF)
    w = torch.randn((N, K), generator=g, device=DEV, dtype=BF) * K ** -0.5
    out = torch.full((M, N), 7.0, dtype=BF, device=DEV)
    qb.qcf_linear(qb.make_desc(inputs.LayerShape(4096, 32, 8, 128, 500000.0, "bf16")), x, M, K, w, N, None, out)
    torch.cuda.synchronize()
    one_rounding(out, x.float() @ w.float().T)


def test_projection_of_very_long_rows():
    """256 weight rows of more than 4 GiB: no tile may address them with 32-bit offsets."""
    say("projection d_model=8500096")
    M, K = 65536, 8500096                # (a size whose cost would speak for the 256 x 256 tiles)
    sh = inputs.LayerShape(K, 2, 1, 128, 500000.0, "bf16")
    g = gen(58)
    x = torch.zeros((2, K), dtype=BF, device=DEV)
    w = torch.zeros((512, K), dtype=BF, device=DEV)
    x[:, -64:] = torch.randn((2, 64), generator=g, device=DEV).to(BF)
    w[:, -64:] = (torch.randn((512, 64), generator=g, device=DEV) * 0.125).to(BF)
    gather = (torch.arange(M, device=DEV) % 2).int()
    q, k, v = (torch.full((M, h, 128), 7.0, dtype=BF, device=DEV) for h in (2, 1, 1))
    qb.qcf_recompute_qkv(qb.make_desc(sh), x, 2, gather, M, w, torch.zeros(M, dtype=torch.int32, device=DEV), q, k, v)
    torch.cuda.synchronize()
    ref = (x[:, -64:].float() @ w[:, -64:].float().T).reshape(2, 4, 128)
    for t, r in ((q, ref[:, :2]), (k, ref[:, 2:3]), (v, ref[:, 3:])):
        one_rounding(t, r[gather.long()])


def test_swiglu_over_the_float_range():
    """Against float64: the argument of the exponential carries a rounding (relative error |g| 2^-24 of the exponential),
    the other operations a few of 2^-24; where the exponential overflows (g < -88.72, a result below 2^-121) it is 0.
    Infinities and NaN as g / (1 + exp(-g)) gives them."""
    g = torch.cat([torch.linspace(-95, 95, 4001), torch.tensor([0.0, -0.0, 1e-30, -1e-30, 3e38, -3e38, -87.4, -88.5, -89.0])])
    g = torch.cat([g, torch.zeros(-g.numel() % 8)])
    F = g.numel()
    out = torch.empty((1, F), dtype=torch.float32, device=DEV)
    desc = qb.make_desc(inputs.LayerShape(256, 4, 2, 64, 10000.0, "f32"))
    qb.qcf_swiglu(desc, torch.cat([g, torch.full((F,), 1.0)]).to(DEV), 1, F, out)
    ref = g.double() / (1.0 + torch.exp(-g.double()))
    err = (out[0].cpu().double() - ref).abs()
    assert bool((err <= (6.0 + 2.0 * g.abs().clamp(max=100.0).double()) * 2.0 ** -24 * ref.abs() + 2.0 ** -121).all())
    special = torch.tensor([float("inf"), -float("inf"), float("nan"), 0.0, 0.0, 0.0, 0.0, 0.0])
    out = torch.empty((1, 8), dtype=torch.float32, device=DEV)
    qb.qcf_swiglu(desc, torch.cat([special, torch.ones(8)]).to(DEV), 1, 8, out)
    got = out[0].cpu()
    assert float(got[0]) == float("inf") and bool(got[1:3].isnan().all()) and bool((got[3:] == 0).all())


def _rotate64(y, pos, base, style):
    """Rotary embedding of y [M, heads, d] in float64."""
    d = y.shape[-1]
    theta = base ** (-2.0 * torch.arange(d // 2, device=y.device, dtype=torch.float64) / d)
    ang = pos.double()[:, None] * theta
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = (y[..., :d // 2], y[..., d // 2:]) if style == 0 else (y[..., 0::2], y[..., 1::2])
    a, b = a.double(), b.double()
    ra, rb = a * c - b * s, b * c + a * s
    return torch.cat([ra, rb], -1) if style == 0 else torch.stack([ra, rb], -1).flatten(-2)


def _rotate(y, pos, base, style):
    return _rotate64(y, pos, base, style).float()


@pytest.mark.parametrize("M,dm,H,Hkv,D,style", [
    (4700, 2048, 32, 8, 128, 0), (4700, 2048, 32, 8, 128, 1), (4700, 2048, 64, 16, 64, 0),   # 256 x 256 tiles
    (4916, 4096, 64, 8, 128, 0), (4916, 4096, 64, 8, 128, 1),                                # rows left for a second launch
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


@pytest.mark.parametrize("M,K,D,style", [(4700, 2048, 128, 0), (4700, 2048, 64, 0), (4700, 2048, 128, 1),      # 256 x 256 tiles
                                         (1500, 2048, 128, 0), (60, 2048, 128, 0), (60, 2048, 64, 1)])      # smaller; split
def test_rotation_at_positions_from_2_24_on(M, K, D, style):
    """Pairs (1, 0) become (cos, sin) of the angle: where one of them is small its bf16 rounding does not hide the angle's
    error.  Bound: one rounding to bf16 plus 3e-7 of a turn."""
    say(f"far positions M={M} D={D} style={style}")
    H, Hkv = 4096 // D, 1024 // D
    sh = inputs.LayerShape(K, H, Hkv, D, 500000.0, "bf16", style)
    x = torch.zeros((M, K), dtype=BF, device=DEV)
    x[:, 5] = 1
    w = torch.zeros((H + 2 * Hkv, D, K), dtype=BF, device=DEV)
    (w[:, :D // 2] if style == 0 else w[:, 0::2])[..., 5] = 1
    pos = torch.randint(1 << 24, (1 << 31) - 1, (M,), generator=gen(53), device=DEV)
    pos[::3] *= -1
    pos[::5] %= 40000                                        # near ones in the same waves
    pos[:4] = torch.tensor([1 << 24, -(1 << 24), (1 << 31) - 1, -(1 << 31)], device=DEV)
    q, k, v = (torch.empty((M, h, D), dtype=BF, device=DEV) for h in (H, Hkv, Hkv))
    qb.qcf_recompute_qkv(qb.make_desc(sh), x, M, None, M, w, pos.int(), q, k, v)
    torch.cuda.synchronize()
    y = torch.zeros((M, 1, D), dtype=torch.float64, device=DEV)
    (y[..., :D // 2] if style == 0 else y[..., 0::2])[:] = 1
    ref = _rotate64(y, pos, 500000.0, style)
    for got in (q, k):
        excess = float(((got.double() - ref).abs() - 2.0 ** -8 * ref.abs()).max())
        assert excess <= 2 * np.pi * 3e-7


@pytest.mark.parametrize("D,style", [(128, 0), (64, 0), (128, 1), (64, 1)])
def test_projection_rounds_alike_in_every_tile(D, style):
    """Without the optional workspace (one contraction per element) a row's bits do not depend on the tile it falls in."""
    say(f"projection bits D={D} style={style}")
    M, dm, H, Hkv = 4700, 2048, 4096 // D, 1024 // D
    sh = inputs.LayerShape(dm, H, Hkv, D, 500000.0, "bf16", style)
    g, desc, lib = gen(56), qb.make_desc(sh), qb.load_library()
    x = torch.randn((M, dm), generator=g, device=DEV, dtype=BF)
    w = torch.randn((sh.qkv_rows, dm), generator=g, device=DEV, dtype=BF) * dm ** -0.5
    pos = torch.randint(0, 40000, (M,), generator=g, device=DEV).int()
    pos[7] = 1 << 25                                         # its wave takes the far path, the other rows keep their bits
    outs = []
    for m in (M, 1229, 300, 60):                             # 256 x 256, 256 x 128, 128 x 128 and 64 x 128 tiles
        q, k, v = (torch.full((m, h, D), 7.0, dtype=BF, device=DEV) for h in (H, Hkv, Hkv))
        assert lib.qcf_recompute_qkv(C.byref(desc), x.data_ptr(), m, None, m, w.data_ptr(), pos.data_ptr(), q.data_ptr(),
                                     k.data_ptr(), v.data_ptr(), None, 0, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        outs.append((q, k, v))
    for o in outs[1:]:
        for a, b in zip(o, outs[0]):
            assert torch.equal(a, b[:a.shape[0]])


@pytest.mark.parametrize("M,dm,H,Hkv", [
    (1300, 4096, 32, 8),             # whole rounds of row tiles, then 20 rows with a split contraction
    (4916, 8192, 64, 8),             # the same, more rows left
    (61, 4096, 32, 8)])              # one launch
@pytest.mark.parametrize("want", ["q", "kv", "v", "scatter"])
def test_projection_outputs_that_are_not_wanted(M, dm, H, Hkv, want):
    """A NULL output is skipped in every launch of a divided product; the others are those of the full call."""
    say(f"projection without some outputs M={M} H={H} want={want}")
    sh = inputs.LayerShape(dm, H, Hkv, 128, 500000.0, "bf16")
    g, desc = gen(52), qb.make_desc(sh)
    x = torch.randn((M, dm), generator=g, device=DEV, dtype=BF)
    w = torch.randn((sh.qkv_rows, dm), generator=g, device=DEV, dtype=BF) * dm ** -0.5
    pos, dst = torch.arange(M, device=DEV).int(), torch.randperm(M, generator=g, device=DEV).int()
    new = lambda: [torch.full((M, h, 128), 7.0, dtype=BF, device=DEV) for h in (H, Hkv, Hkv)]
    full, part = new(), new()
    qb.qcf_recompute_qkv(desc, x, M, None, M, w, pos, *full)
    if want == "scatter":
        kf, vf = torch.full_like(part[1], 7.0), torch.full_like(part[2], 7.0)
        qb.qcf_recompute_qkv_scatter(desc, x, M, None, M, w, pos, None, part[1], part[2], dst, kf, vf, M)
        got, kept = (1, 2), (0,)
    else:
        got = {"q": (0,), "kv": (1, 2), "v": (2,)}[want]
        kept = tuple(i for i in range(3) if i not in got)
        qb.qcf_recompute_qkv(desc, x, M, None, M, w, pos, *(part[i] if i in got else None for i in range(3)))
    torch.cuda.synchronize()
    for i in got:
        assert torch.equal(part[i], full[i])
    for i in kept:
        assert bool((part[i] == 7.0).all())
    if want == "scatter":
        assert torch.equal(kf[dst.long()], full[1]) and torch.equal(vf[dst.long()], full[2])


def _attention64(q, k, v, pos, scale):
    """Plain float64 attention of rows q [n, H, d] over k, v [T, Hkv, d]; row i sees tokens <= pos[i]."""
    G = q.shape[1] // k.shape[1]
    kk, vv = (t.double().repeat_interleave(G, dim=1).transpose(0, 1) for t in (k, v))
    s = q.double().transpose(0, 1) @ kk.transpose(1, 2) * scale
    s.masked_fill_(torch.arange(k.shape[0], device=k.device)[None, None] > pos.long()[None, :, None], -float("inf"))
    p = torch.softmax(s, -1)
    return (p @ vv).transpose(0, 1), torch.logsumexp(s, -1).T


@pytest.mark.parametrize("H,Hkv,ctx,sel,with_ws", [
    (8, 2, [300, 1, 64, 1025], [45, 1, 10, 150], True),       # ragged requests
    (32, 8, [4099], [615], True),                             # key ranges split over workgroups, fp32 partials
    (32, 8, [4099], [615], False),                            # the same without the optional workspace
    (4, 4, [2048], [33], True), (16, 1, [63], [63], True)])   # one head per group; sixteen
def test_attention_of_64_wide_heads(H, Hkv, ctx, sel, with_ws):
    """bf16 rows over bf16 keys and values: only the stored result is rounded to bf16."""
    say(f"attention d=64 H={H} Hkv={Hkv} ctx={ctx} sel={sel} ws={with_ws}")
    sh = inputs.LayerShape(2048, H, Hkv, 64, 10000.0, "bf16")
    g, desc = gen(46), qb.make_desc(sh)
    T, N = sum(ctx), sum(sel)
    q = torch.randn((N, H, 64), generator=g, device=DEV, dtype=BF) * 2
    k, v = (torch.randn((T, Hkv, 64), generator=g, device=DEV, dtype=BF) for _ in range(2))
    pos = [torch.sort(torch.randperm(t, generator=g, device=DEV)[:n])[0].int() for t, n in zip(ctx, sel)]
    so, co = i64(np.concatenate([[0], np.cumsum(sel)])), i64(np.concatenate([[0], np.cumsum(ctx)]))
    o, lse = torch.full((N, H, 64), 7.0, dtype=BF, device=DEV), torch.full((N, H), 7.0, device=DEV)
    p = torch.cat(pos)
    if with_ws:
        qb.qcf_recompute_attn(desc, len(ctx), q, p, so, N, k, v, co, T, None, o, lse)
    else:
        assert qb.load_library().qcf_recompute_attn(
            C.byref(desc), len(ctx), q.data_ptr(), p.data_ptr(), so.data_ptr(), N, k.data_ptr(), v.data_ptr(), co.data_ptr(),
            T, None, o.data_ptr(), lse.data_ptr(), None, 0, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    s0 = c0 = 0
    for t, n, ps in zip(ctx, sel, pos):
        ro, rl = _attention64(q[s0:s0 + n], k[c0:c0 + t], v[c0:c0 + t], ps, 0.125)
        one_rounding(o[s0:s0 + n], ro.float())
        assert float((lse[s0:s0 + n].double() - rl).abs().max()) < 2e-5
        s0, c0 = s0 + n, c0 + t


@pytest.mark.parametrize("D,H,Hkv,ctx,sel", [
    (128, 32, 8, [731], [110]), (128, 32, 8, [600, 30, 1500], [40, 3, 90]), (128, 4, 4, [1100], [300]), (128, 32, 1, [2000], [5]),
    (64, 32, 8, [731], [110]), (64, 32, 8, [600, 30, 1500], [40, 3, 90]),      # units that all start at once: no plan
    (128, 32, 8, [6000], [300])])                                                # more than that: sorted by length
def test_attention_of_split_row_blocks(D, H, Hkv, ctx, sel):
    """Key ranges cut into segments, with and without the plan kernel; some rows see nothing."""
    say(f"split attention D={D} H={H} ctx={ctx} sel={sel}")
    sh = inputs.LayerShape(2048, H, Hkv, D, 10000.0, "bf16")
    g, desc = gen(60), qb.make_desc(sh)
    T, N = sum(ctx), sum(sel)
    assert qb.qcf_recompute_attn_workspace_bytes(desc, len(ctx), N, T) > 0
    q = torch.randn((N, H, D), generator=g, device=DEV, dtype=BF)
    k, v = (torch.randn((T, Hkv, D), generator=g, device=DEV, dtype=BF) for _ in range(2))
    pos = [torch.sort(torch.randperm(t, generator=g, device=DEV)[:n])[0].int() for t, n in zip(ctx, sel)]
    pos[0][:2] = -1                                          # sees nothing
    so, co = i64(np.concatenate([[0], np.cumsum(sel)])), i64(np.concatenate([[0], np.cumsum(ctx)]))
    o, lse = torch.full((N, H, D), 7.0, dtype=BF, device=DEV), torch.full((N, H), 7.0, device=DEV)
    qb.qcf_recompute_attn(desc, len(ctx), q, torch.cat(pos), so, N, k, v, co, T, None, o, lse)
    torch.cuda.synchronize()
    s0 = c0 = 0
    for t, n, ps in zip(ctx, sel, pos):
        ro, rl = _attention64(q[s0:s0 + n], k[c0:c0 + t], v[c0:c0 + t], ps, D ** -0.5)
        none = ps < 0
        ro[none] = 0.0
        got, glse = o[s0:s0 + n], lse[s0:s0 + n].double()
        # d = 128: probabilities and partial outputs are bf16, values up to about 4
        assert float((got.double() - ro).abs().max()) < (2e-2 if D == 128 else 1.6e-2)
        assert bool((glse[none] == -float("inf")).all()) and float((glse - rl)[~none].abs().max()) < 2e-5
        s0, c0 = s0 + n, c0 + t


@pytest.mark.parametrize("T,n", [(200, 40), (4099, 615)])      # whole row blocks; split ones
def test_attention_of_64_wide_heads_infinite_values(T, n):
    """An infinite value reaches the rows that see its token, as an infinity, and no others."""
    say(f"attention d=64 infinite value T={T}")
    sh = inputs.LayerShape(2048, 32, 8, 64, 10000.0, "bf16")
    g = gen(47)
    q = torch.randn((n, 32, 64), generator=g, device=DEV, dtype=BF)
    k, v = (torch.randn((T, 8, 64), generator=g, device=DEV, dtype=BF) for _ in range(2))
    at = T - T // 3
    pos = torch.sort(torch.randperm(T, generator=g, device=DEV)[:n])[0].int()
    o = torch.empty((n, 32, 64), dtype=BF, device=DEV)
    clean = _attention64(q, k, v, pos, 0.125)[0]
    v[at, :, 5] = float("inf")
    qb.qcf_recompute_attn(qb.make_desc(sh), 1, q, pos, i64([0, n]), n, k, v, i64([0, T]), T, None, o, None)
    torch.cuda.synchronize()
    sees = (pos >= at)[:, None].expand(-1, 32)
    ref = clean.float()
    assert bool((o[:, :, 5][sees] == float("inf")).all())
    keep = torch.ones_like(ref, dtype=torch.bool)
    keep[:, :, 5] = ~sees
    one_rounding(o[keep], ref[keep])


@pytest.mark.parametrize("T,n", [(200, 40), (4099, 615)])      # whole row blocks; split ones
@pytest.mark.parametrize("what", ["nan key", "nan values", "both infinities", "minus infinity", "large", "no weight", "huge logits"])
def test_attention_of_64_wide_heads_special_values(T, n, what):
    """What a row does not see leaves no trace; what it sees gives NaN, an infinity or (large finite values) a finite
    number as the sum over its visible tokens does, and a NaN log-sum-exp where a logit is NaN."""
    say(f"attention d=64 {what} T={T}")
    sh = inputs.LayerShape(2048, 32, 8, 64, 10000.0, "bf16")
    g, inf, nan = gen(55), float("inf"), float("nan")
    q = torch.randn((n, 32, 64), generator=g, device=DEV, dtype=BF)
    k, v = (torch.randn((T, 8, 64), generator=g, device=DEV, dtype=BF) for _ in range(2))
    pos = torch.sort(torch.randperm(T, generator=g, device=DEV)[:n])[0].int()
    pos[0] = 0
    at = T // 3
    if what == "large":                  # logits that rise by 5 after the first tokens: less than the reference point may lag
        q[:], k[:], v[:] = 1.0, 0.0, 0.0
        k[at:, :, 0] = 40.0
        v[at, :, 7] = 3.0e38
    if what == "no weight":              # the first token's logit is -infinity, and row 0 sees nothing else
        q[:, :, 9] = q[:, :, 9].abs() + 0.5
        k[0, :, 9] = -inf
    if what == "huge logits":            # one token takes all of a row's weight
        q, k = q * 1e18, k * 1e18
    ro, rl = _attention64(q, k, v, pos, 0.125)
    ref, lse_ref = ro.float(), rl.float()
    sees = pos >= at
    if what == "nan key":
        k[at, :, 11] = nan
        ref[sees], lse_ref[sees] = nan, nan
    elif what == "nan values":
        v[at:] = nan
        ref[sees] = nan
    elif what == "both infinities":
        v[at, :, 5], v[at + 3, :, 5], v[at + 3, :, 6] = inf, -inf, -inf
        ref[:, :, 5][pos >= at] = inf
        ref[:, :, 5][pos >= at + 3] = nan
        ref[:, :, 6][pos >= at + 3] = -inf
    elif what == "minus infinity":
        v[at, 3, 63] = -inf
        ref[:, 12:16, 63][sees] = -inf
    elif what == "no weight":
        ref[pos == 0], lse_ref[pos == 0] = nan, nan
    elif what == "large":
        assert bool(ref.isfinite().all()) and float(ref.max()) > 1e35
    o, lse = torch.full((n, 32, 64), 7.0, dtype=BF, device=DEV), torch.full((n, 32), 7.0, device=DEV)
    qb.qcf_recompute_attn(qb.make_desc(sh), 1, q, pos, i64([0, n]), n, k, v, i64([0, T]), T, None, o, lse)
    torch.cuda.synchronize()
    of = o.float()
    assert torch.equal(of.isnan(), ref.isnan()) and torch.equal(lse.isnan(), lse_ref.isnan())
    assert torch.equal(of.isinf(), ref.isinf()) and torch.equal(of[ref.isinf()], ref[ref.isinf()])
    fin = ref.isfinite()
    err = (of[fin] - ref[fin]).abs() - 2.0 ** -8 * ref[fin].abs()
    assert float(err.max()) <= 2e-4
    fin = lse_ref.isfinite()
    # (huge: 64 products of size up to 2e37 / 8, each sum rounded to 2^-24 of at most 1e37)
    assert float((lse[fin] - lse_ref[fin]).abs().max()) < (64 * 2.0 ** -24 * 1e37 if what == "huge logits" else 2e-5)


@pytest.mark.parametrize("H,Hkv,ctx,probes,limit", [
    (32, 8, [4099], [40], False), (8, 2, [300, 1, 64, 1025, 256], [5, 3, 0, 17, 30], False),
    (8, 4, [700], [33], True),
    (32, 8, [9000], [40], False), (8, 2, [300, 1, 2000], [90, 3, 100], True)])                  # several blocks of rows
def test_scores_of_64_wide_heads(H, Hkv, ctx, probes, limit):
    say(f"scores d=64 H={H} Hkv={Hkv} ctx={ctx} probes={probes}")
    sh = inputs.LayerShape(2048, H, Hkv, 64, 10000.0, "bf16")
    g = gen(48)
    T, R = sum(ctx), sum(probes)
    q = torch.randn((R, H, 64), generator=g, device=DEV, dtype=BF) * 2
    k = torch.randn((T, Hkv, 64), generator=g, device=DEV, dtype=BF)
    lim = torch.cat([torch.randint(1, t + 1, (r,), generator=g, device=DEV) for t, r in zip(ctx, probes)]).int()
    po, co = i64(np.concatenate([[0], np.cumsum(probes)])), i64(np.concatenate([[0], np.cumsum(ctx)]))
    score = torch.full((T,), 7.0, device=DEV)
    qb.qcf_score(qb.make_desc(sh), len(ctx), q, po, R, k, co, T, lim if limit else None, score)
    torch.cuda.synchronize()
    r0 = c0 = 0
    for t, r in zip(ctx, probes):
        kk = k[c0:c0 + t].double().repeat_interleave(H // Hkv, dim=1).permute(1, 2, 0)
        s = q[r0:r0 + r].double().transpose(0, 1) @ kk * 0.125
        if limit:
            s.masked_fill_(torch.arange(t, device=DEV)[None, None] >= lim[r0:r0 + r].long()[None, :, None], -float("inf"))
        ref = torch.softmax(s, -1).mean((0, 1)) if r else torch.zeros(t, dtype=torch.float64, device=DEV)
        # 32-bit logits of magnitude up to 60, exponentials and sums
        assert bool(((score[c0:c0 + t].double() - ref).abs() <= 3e-5 * ref + 1e-12).all())
        r0, c0 = r0 + r, c0 + t


@pytest.mark.parametrize("T,R", [(300, 12), (4099, 40), (1000, 100)])
@pytest.mark.parametrize("what", ["nan key", "nan key beyond the limits", "infinite key", "one token at minus infinity",
                                  "no weight", "a row that sees nothing", "large logits", "huge logits"])
def test_scores_of_64_wide_heads_special_values(T, R, what):
    """A NaN or infinite logit makes its row's softmax, and so every score, NaN, unless no row sees it; so does a row whose
    visible logits are all -infinity.  Large logits: the error of a float32 logit (2^-24 of it, and of its 64 products)."""
    say(f"scores d=64 {what} T={T}")
    H, Hkv = 8, 2
    sh = inputs.LayerShape(512, H, Hkv, 64, 10000.0, "bf16")
    g, inf = gen(61), float("inf")
    q = torch.randn((R, H, 64), generator=g, device=DEV).to(BF)
    k = torch.randn((T, Hkv, 64), generator=g, device=DEV).to(BF)
    q[:, :, 3] = q[:, :, 3].abs() + 0.1
    lim = None
    clean = k.clone()
    if what == "nan key":
        k[T // 2, 1, 3] = float("nan")
    elif what == "nan key beyond the limits":
        k[T // 2, 1, 3] = float("nan")
        lim = torch.full((R,), T // 2, dtype=torch.int32, device=DEV)
    elif what == "infinite key":
        k[T // 2, 0, 3] = inf
    elif what == "one token at minus infinity":
        k[T // 2, :, 3] = -inf
        clean = k
    elif what == "no weight":
        k[:, :, 3] = -inf
    elif what == "a row that sees nothing":
        lim = torch.full((R,), T // 3, dtype=torch.int32, device=DEV)
        lim[:3] = 0
    else:
        q *= 100 if what == "large logits" else 1e18
        k *= 1 if what == "large logits" else 1e18
        clean = k
    score = torch.full((T,), 7.0, device=DEV)
    qb.qcf_score(qb.make_desc(sh), 1, q, i64([0, R]), R, k, i64([0, T]), T, lim, score)
    torch.cuda.synchronize()
    if what in ("nan key", "infinite key", "no weight"):
        assert bool(score.isnan().all())
        return
    s = q.double().transpose(0, 1) @ clean.double().repeat_interleave(H // Hkv, dim=1).permute(1, 2, 0) * 0.125
    if lim is not None:
        s.masked_fill_(torch.arange(T, device=DEV)[None, None] >= lim.long()[None, :, None], -inf)
    ref = torch.softmax(s, -1).nan_to_num(0.0).mean((0, 1))
    if what == "large logits":
        # random roundings: the error of the sum over rows stays near 1e-6; one rounded log-sum-exp gave 4e-6 to 9e-6
        assert float((score.double() - ref).norm() / ref.norm()) < 3e-6
    else:
        assert bool(((score.double() - ref).abs() <= 3e-5 * ref + 1e-12).all())


def test_scores_of_64_wide_heads_on_many_streams():
    """Calls that overlap on more streams than the library has counter sets: each gets what it gets alone, bit for bit."""
    say("scores d=64 on 12 streams")
    sh = inputs.LayerShape(2048, 32, 8, 64, 10000.0, "bf16")
    g, desc, T, R, n = gen(54), qb.make_desc(sh), 4099, 40, 12
    q = [torch.randn((R, 32, 64), generator=g, device=DEV, dtype=BF) for _ in range(n)]
    k = [torch.randn((T, 8, 64), generator=g, device=DEV, dtype=BF) for _ in range(n)]
    po, co = i64([0, R]), i64([0, T])
    need = qb.qcf_score_workspace_bytes(desc, 1, R, T)
    ws = [torch.empty(need, dtype=torch.uint8, device=DEV) for _ in range(n)]
    alone, many = (torch.empty((n, T + 1), device=DEV)[:, :T] for _ in range(2))       # (rows 16-byte aligned)
    assert alone.stride(0) % 4 == 0
    for i in range(n):
        qb.qcf_score(desc, 1, q[i], po, R, k[i], co, T, None, alone[i], ws[i])
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(n)]
    for _ in range(4):
        many.fill_(7.0)
        torch.cuda.synchronize()
        for i in range(n):
            with torch.cuda.stream(streams[i]):
                qb.qcf_score(desc, 1, q[i], po, R, k[i], co, T, None, many[i], ws[i])
        torch.cuda.synchronize()
        assert torch.equal(alone, many)


@pytest.mark.parametrize("dtype,M,K,N", [("f32", 1, 8, 8), ("f32", 77, 256, 512), ("f32", 17, 264, 40), ("f32", 1100, 72, 1032),
                                         ("bf16", 33, 520, 48), ("bf16", 5, 24, 16)])
def test_general_product_tiles(dtype, M, K, N):
    """Both tiles of the general product, edges included."""
    say(f"general product {dtype} M={M} K={K} N={N}")
    g = gen(49)
    dt = inputs.torch_dtype(dtype)
    x = torch.randn((M, K), generator=g, device=DEV).to(dt)
    w = (torch.randn((N, K), generator=g, device=DEV) * K ** -0.5).to(dt)
    out = torch.full((M, N), 7.0, dtype=dt, device=DEV)
    desc = qb.make_desc(inputs.LayerShape(256, 4, 2, 64, 10000.0, dtype))
    qb.qcf_linear(desc, x, M, K, w, N, None, out)
    torch.cuda.synchronize()
    ref = (x.double() @ w.double().T).float()
    if dtype == "bf16":
        one_rounding(out, ref)
    else:
        assert float((out - ref).abs().max()) < 1e-5          # 32-bit sums of up to 260 products of size K^-1/2


@pytest.mark.parametrize("D,T,n", [(64, 257, 40), (128, 300, 31), (64, 31, 31), (128, 1, 1)])
def test_f32_attention_general(D, T, n):
    """Tiles of 256 tokens and the value loop's remainders, against float64."""
    say(f"f32 attention D={D} T={T}")
    g = gen(50)
    q = torch.randn((n, 4, D), generator=g, device=DEV)
    k, v = (torch.randn((T, 2, D), generator=g, device=DEV) for _ in range(2))
    pos = torch.sort(torch.randperm(T, generator=g, device=DEV)[:n])[0].int()
    o, lse = torch.full((n, 4, D), 7.0, device=DEV), torch.full((n, 4), 7.0, device=DEV)
    desc = qb.make_desc(inputs.LayerShape(256, 4, 2, D, 10000.0, "f32"))
    qb.qcf_recompute_attn(desc, 1, q, pos, i64([0, n]), n, k, v, i64([0, T]), T, None, o, lse)
    torch.cuda.synchronize()
    ro, rl = _attention64(q, k, v, pos, D ** -0.5)
    assert float((o.double() - ro).abs().max()) < 1e-5
    assert float((lse.double() - rl).abs().max()) < 1e-5


@pytest.mark.parametrize("dtype,H,Hkv,D", [("f32", 8, 2, 64), ("f32", 8, 4, 128), ("bf16", 12, 4, 128), ("bf16", 12, 4, 64)])
@pytest.mark.parametrize("T", [1, 65, 257, 600])
def test_generic_attention_of_many_rows(dtype, H, Hkv, D, T):
    """Launches of many workgroups take another instance with the same sums in the same order: a row's bits are those of a launch of
    few, which the tests above compare with float64."""
    say(f"generic attention of many rows {dtype} D={D} T={T}")
    g, dt, n = gen(65), inputs.torch_dtype(dtype), 200
    q = torch.randn((n, H, D), generator=g, device=DEV).to(dt)
    k, v = (torch.randn((T, Hkv, D), generator=g, device=DEV).to(dt) for _ in range(2))
    pos = torch.randint(-1, T, (n,), generator=g, device=DEV).int()
    desc = qb.make_desc(inputs.LayerShape(256, H, Hkv, D, 10000.0, dtype))

    def attend(rows):
        o, lse = torch.full((rows, H, D), 7.0, device=DEV, dtype=dt), torch.full((rows, H), 7.0, device=DEV)
        qb.qcf_recompute_attn(desc, 1, q, pos, i64([0, rows]), rows, k, v, i64([0, T]), T, None, o, lse)
        return o, lse

    (many, many_lse), (few, few_lse) = attend(n), attend(20)
    torch.cuda.synchronize()
    assert torch.equal(many[:20], few) and torch.equal(many_lse[:20], few_lse)
    ro, rl = _attention64(q, k, v, pos, D ** -0.5)
    see = pos >= 0
    assert float((many.double() - ro)[see].abs().max()) < (1e-5 if dtype == "f32" else 2e-2) and bool((many[~see] == 0).all())
    assert float((many_lse.double() - rl)[see].abs().max()) < 1e-5


@pytest.mark.parametrize("lens", [[300], [1, 1021], [4094], [5000, 3190], [1, 1024, 1025, 3], [4096, 4097, 8192, 8193, 16384], [16385, 7, 32768], [32769, 1023, 40001]])
def test_select_keys_per_thread(lens):
    """Every number of keys per thread, requests that start at any alignment, ties: exactly the N largest, ties to the
    lower index, ascending."""
    say(f"select {lens}")
    g = gen(51)
    lens = [2] + lens                                        # (shifts the starts)
    T = sum(lens)
    score = torch.exp(torch.randn(T, generator=g, device=DEV) * 2)
    score[::7] = score[0]                                    # ties
    counts = [max(1, int(0.15 * n)) for n in lens]
    co, so = i64(np.concatenate([[0], np.cumsum(lens)])), i64(np.concatenate([[0], np.cumsum(counts)]))
    N = sum(counts)
    idx, row, pos = (torch.full((N,), -7, dtype=torch.int32, device=DEV) for _ in range(3))
    qb.qcf_select(len(lens), score, co, T, so, N, None, idx, row, pos)
    torch.cuda.synchronize()
    c0 = s0 = 0
    for n, m in zip(lens, counts):
        ref = torch.sort(torch.sort(score[c0:c0 + n], descending=True, stable=True)[1][:m])[0].int()
        assert torch.equal(idx[s0:s0 + m], ref) and torch.equal(pos[s0:s0 + m], ref) and torch.equal(row[s0:s0 + m], ref + c0)
        c0, s0 = c0 + n, s0 + m


@pytest.mark.parametrize("D,T,R", [(64, 1, 1), (64, 3, 2), (64, 255, 5), (64, 257, 3), (64, 2048, 2), (64, 2049, 2), (128, 1, 3), (128, 127, 20), (128, 2047, 3), (128, 4100, 2)])
def test_f32_scoring_rows(D, T, R):
    """Tokens per load and per wave, a row in LDS and in the workspace, rows that see part of the context: against float64.
    Bound: worst case of the dot products' rounding in the exponent, of the sums over a row and over the rows."""
    say(f"f32 scoring D={D} T={T} R={R}")
    g = gen(61)
    H, Hkv = 4, 2
    q, k = torch.randn((R, H, D), generator=g, device=DEV), torch.randn((T, Hkv, D), generator=g, device=DEV)
    limit = torch.randint(1, T + 1, (R,), generator=g, device=DEV).int()
    desc = qb.make_desc(inputs.LayerShape(256, H, Hkv, D, 10000.0, "f32"))
    kk = k.double().repeat_interleave(H // Hkv, 1)
    logits = torch.einsum("rhd,thd->rht", q.double().cpu(), kk.cpu()) * D ** -0.5
    size = float(torch.einsum("rhd,thd->rht", q.double().abs().cpu(), kk.abs().cpu()).max()) * D ** -0.5
    bound = 2.0 ** -24 * (2 * (D + 4) * size + T + R * H + 64)
    for lim in (None, limit):
        out = torch.full((T,), 7.0, device=DEV)
        if lim is None:
            qb.qcf_score(desc, 1, q, i64([0, R]), R, k, i64([0, T]), T, None, out)
            p = torch.softmax(logits, -1)
        else:
            qb.qcf_score(desc, 1, q, i64([0, R]), R, k, i64([0, T]), T, lim, out)
            p = torch.softmax(logits.masked_fill(torch.arange(T)[None, None] >= lim.cpu()[:, None, None], -torch.inf), -1)
        torch.cuda.synchronize()
        ref = p.mean((0, 1))
        assert bool(((out.double().cpu() - ref).abs() <= bound * ref).all()), float(((out.double().cpu() - ref).abs() / ref.clamp_min(1e-30)).max())


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("T,R", [
    ([1, 300, 64, 0, 513, 30, 2100], [3, 1, 20, 2, 5, 0, 2]),        # 430 tokens on average: fewer threads to a row; one row in the workspace
    ([64] * 9, [4] * 9), ([600, 425], [3, 2])])                     # 512.5: as a single request
def test_f32_scoring_of_several_requests(D, T, R):
    """Bounds as above, of the longest request."""
    say(f"f32 scoring D={D} of {T} tokens")
    g, H, Hkv, B = gen(66), 4, 2, len(T)
    q, k = torch.randn((sum(R), H, D), generator=g, device=DEV), torch.randn((sum(T), Hkv, D), generator=g, device=DEV)
    off = lambda n: [0] + list(np.cumsum(n))
    po, co = off(R), off(T)
    out = torch.full((sum(T),), 7.0, device=DEV)
    desc = qb.make_desc(inputs.LayerShape(256, H, Hkv, D, 10000.0, "f32"))
    qb.qcf_score(desc, B, q, i64(po), sum(R), k, i64(co), sum(T), None, out)
    torch.cuda.synchronize()
    for b in range(B):
        qq, kk = q[po[b]:po[b + 1]].double().cpu(), k[co[b]:co[b + 1]].double().cpu().repeat_interleave(H // Hkv, 1)
        got = out[co[b]:co[b + 1]].double().cpu()
        if not R[b] or not T[b]:
            assert bool((got == 0).all())
            continue
        ref = torch.softmax(torch.einsum("rhd,thd->rht", qq, kk) * D ** -0.5, -1).mean((0, 1))
        size = float(torch.einsum("rhd,thd->rht", qq.abs(), kk.abs()).max()) * D ** -0.5
        assert bool(((got - ref).abs() <= 2.0 ** -24 * (2 * (D + 4) * size + T[b] + R[b] * H + 64) * ref).all()), b


@pytest.mark.parametrize("T", [127, 129, 1000, 1025, 3001, 9001, 40001])
def test_select_crowded_bins_and_extreme_keys(T):
    """Keys that crowd one bin, the whole range of 32 bits, the NaN of the lowest key, more outputs than leave together:
    the N largest by their order-preserving keys, ties to the lower index."""
    say(f"select extremes {T}")
    rng = np.random.default_rng(T)
    low = np.array([0xFFFFFFFF], np.uint32).view(np.float32)[0]
    crowd = (0x3F000000 + rng.integers(0, max(T // 3, 2), T)).astype(np.uint32).view(np.float32)
    crowd[T // 2] = 1e-30
    wide = rng.integers(0, 2 ** 32, T, dtype=np.uint64).astype(np.uint32).view(np.float32)
    wide[1::5] = wide[0]
    lowest = np.where(rng.random(T) < 0.3, low, wide).astype(np.float32)
    lowest.view(np.uint32)[3] = 0xFFFFFFFF
    for s in (crowd, wide, lowest, rng.choice(np.float32([np.inf, -np.inf, 0.0, -0.0, 2.0]), T)):
        u = s.view(np.uint32).copy()
        u[u == 0x80000000] = 0
        key = np.where(u >> 31 != 0, ~u, u | 0x80000000).astype(np.int64)
        order = np.argsort(-key, kind="stable")
        for n in sorted({1, T // 7, T // 2, T - 2, T - 1}):
            want = np.sort(order[:n]).astype(np.int32)
            d = torch.from_numpy(s.view(np.int32).copy()).to(DEV).view(torch.float32)
            idx, row, pos = (torch.full((n,), -7, dtype=torch.int32, device=DEV) for _ in range(3))
            qb.qcf_select(1, d, i64([0, T]), T, i64([0, n]), n, None, idx, row, pos)
            torch.cuda.synchronize()
            assert all(np.array_equal(x.cpu().numpy(), want) for x in (idx, row, pos)), (T, n)


@pytest.mark.parametrize("T", [3840, 3841, 7936, 7937, 16128, 16129, 20000, 32512, 32513])
def test_select_rows_that_are_not_there(T):
    """The edges between requests in which every wave has all its rows and those in which some lack one: keys of both signs, all equal,
    and the extremes of above."""
    say(f"select rows {T}")
    test_select_crowded_bins_and_extreme_keys(T)
    n = int(0.15 * T)
    for s in (torch.randn(T, generator=gen(64), device=DEV), torch.zeros(T, device=DEV)):
        out = [torch.full((n,), -7, dtype=torch.int32, device=DEV) for _ in range(3)]
        qb.qcf_select(1, s, i64([0, T]), T, i64([0, n]), n, None, *out)
        ref = torch.sort(torch.sort(s, descending=True, stable=True)[1][:n])[0].int()
        assert all(torch.equal(x, ref) for x in out)


def test_select_of_many_outputs_reads_the_scores_once_more():
    """A million keys: half of them selected takes no more passes over the keys than 8192, only more stores.  (With a pass per 8192
    outputs 18 times as long; the line is far from that and from 1.)"""
    say("select half of a million")
    T = 1 << 20
    score = torch.exp(torch.randn(T, generator=gen(63), device=DEV))

    def ms(n):
        out = [torch.empty(n, dtype=torch.int32, device=DEV) for _ in range(3)]
        call = lambda: qb.qcf_select(1, score, i64([0, T]), T, i64([0, n]), n, None, *out)
        call()
        torch.cuda.synchronize()
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            call()
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        ref = torch.sort(torch.sort(score, descending=True, stable=True)[1][:n])[0].int()
        assert all(torch.equal(x, ref) for x in out), n
        return best

    assert ms(T // 2) < 4 * ms(8192)


def test_anchor_extraction_is_refused_under_capture():
    """Its offsets come from a pinned block that is handed back after the call; a replay would read whatever is there."""
    say("anchors under capture")
    sh = inputs.LayerShape(4096, 32, 8, 128, 500000.0, "bf16")
    k, v = (torch.randn((96, 8, 128), generator=gen(59), device=DEV, dtype=BF) for _ in range(2))
    desc, graph = qb.make_desc(sh), torch.cuda.CUDAGraph()
    want = pipeline.extract_anchors(desc, k, v, [64, 32], [4, 2])        # (allocations are warm, the pinned block is free again)
    torch.cuda.synchronize()
    refused = False
    with torch.cuda.graph(graph):
        t = k * 1.0
        try:
            pipeline.extract_anchors(desc, k, v, [64, 32], [4, 2])
        except RuntimeError:
            refused = True
    assert refused
    got = pipeline.extract_anchors(desc, k, v, [64, 32], [4, 2])
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("many", [False, True])          # 512 and 256 threads to a workgroup
@pytest.mark.parametrize("H,Hkv,D,T", [(4, 2, 64, 511), (4, 2, 128, 513), (3, 3, 64, 257), (6, 2, 128, 64), (8, 2, 64, 1025), (5, 1, 128, 1)])
def test_f32_attention_by_lanes(H, Hkv, D, T, many):
    """Tokens shared by the lanes of a wave, pairs of heads (even groups) and single ones; edges of tiles of 256 and 512 tokens, rows
    that see one token, all of them and none, a request without rows between two others."""
    n = 600 if many else 7
    say(f"f32 attention by lanes H={H}/{Hkv} D={D} T={T} rows={n}")
    g = gen(91)
    lens, rows = [T, 5, 2 * T], [n, 0, 3]
    off = lambda v: torch.tensor([sum(v[:i]) for i in range(len(v) + 1)], dtype=torch.int64, device=DEV)
    q = torch.randn((sum(rows), H, D), generator=g, device=DEV)
    k, v = (torch.randn((sum(lens), Hkv, D), generator=g, device=DEV) for _ in range(2))
    pos = torch.cat([torch.randint(0, T, (n,), generator=g, device=DEV), torch.randint(0, 2 * T, (3,), generator=g, device=DEV)]).int()
    pos[0], pos[1], pos[2], pos[3] = 0, T - 1, -1, T + 100            # (one token, all, none, all)
    desc = qb.make_desc(inputs.LayerShape(256, H, Hkv, D, 10000.0, "f32"))
    o, lse = torch.full_like(q, 7.0), torch.full((sum(rows), H), 7.0, device=DEV)
    qb.qcf_recompute_attn(desc, 3, q, pos, off(rows), sum(rows), k, v, off(lens), sum(lens), None, o, lse)
    torch.cuda.synchronize()
    for lo, hi, c0, c1 in ((0, n, 0, T), (n, n + 3, T + 5, 3 * T + 5)):
        kk, vv = (x[c0:c1].double().repeat_interleave(H // Hkv, 1) for x in (k, v))
        s = q[lo:hi].double().transpose(0, 1) @ kk.permute(1, 2, 0).contiguous() / math.sqrt(D)
        s.masked_fill_(torch.arange(c1 - c0, device=DEV) > pos[lo:hi].long()[None, :, None], -math.inf)
        ref = (torch.softmax(s, -1).nan_to_num(0.0) @ vv.transpose(0, 1).contiguous()).transpose(0, 1)
        # 32-bit logits of D terms (an error of about 1e-6 in the exponent) and sums of up to 2050 positive weights
        assert float((o[lo:hi].double() - ref).abs().max()) < 1e-5
        want, got = torch.logsumexp(s, -1).transpose(0, 1), lse[lo:hi].double()
        assert bool((((got - want).abs() < 1e-5) | ((want == -math.inf) & (got == -math.inf))).all())


@pytest.mark.parametrize("H,Hkv,D", [(4, 2, 64), (3, 3, 64), (8, 2, 128), (5, 1, 128)])
@pytest.mark.parametrize("T", [1, 5, 63, 64, 65, 200, 511, 513, 1100])
def test_f32_attention_has_one_order_of_sums(H, Hkv, D, T):
    """A row has the same bits in a call of 7 rows (512 threads to a workgroup) as among 600 (256 threads), whatever share of a tile's
    tokens a wave gets."""
    say(f"f32 attention, 7 rows and 600, H={H}/{Hkv} D={D} T={T}")
    g = gen(92)
    n = 600
    q = torch.randn((n, H, D), generator=g, device=DEV)
    k, v = (torch.randn((T, Hkv, D), generator=g, device=DEV) for _ in range(2))
    pos = torch.randint(0, T, (n,), generator=g, device=DEV).int()
    pos[0], pos[1], pos[2] = 0, T - 1, T + 7
    desc = qb.make_desc(inputs.LayerShape(256, H, Hkv, D, 10000.0, "f32"))
    off = lambda rows: torch.tensor([0, rows], dtype=torch.int64, device=DEV)

    def attend(rows):
        o, lse = torch.full((rows, H, D), 7.0, device=DEV), torch.full((rows, H), 7.0, device=DEV)
        qb.qcf_recompute_attn(desc, 1, q[:rows].contiguous(), pos[:rows].contiguous(), off(rows), rows, k, v, off(T), T, None, o, lse)
        torch.cuda.synchronize()
        return o, lse

    for few, many in zip(attend(7), attend(n)):
        assert torch.equal(few.view(torch.int32), many[:7].view(torch.int32))
