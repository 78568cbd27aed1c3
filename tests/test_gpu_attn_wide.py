"""Attention of 128-wide heads with 256 rows to a workgroup: launches long enough for it, edges of blocks and tiles."""
import math

import pytest
import torch

from paper_2604_08585_amd import binding as qb
from paper_2604_08585_amd import inputs
import host_rules
from gpu_util import DEV, i64

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


def say(msg):
    print(msg, flush=True)


def _case(seed, H, Hkv, T, sel, q_std=1.0, pos0=None, pos=None):
    """Requests of T[b] tokens, sel[b] rows each, against float64.  Probabilities are rounded to bf16 once and so is the
    result.  bf16 has eight significant bits, so rounding is off by at most 2^-8 of the value (half of 2^-7):
    |error| <= 2^-8 sum p |v| + 2^-8 |o|, and a little for the 32-bit sums."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    off = lambda v: [sum(v[:i]) for i in range(len(v) + 1)]
    oc, os_ = off(T), off(sel)
    q = (torch.randn((sum(sel), H, 128), generator=g, device=DEV) * q_std).to(BF)
    k, v = (torch.randn((sum(T), Hkv, 128), generator=g, device=DEV, dtype=BF) for _ in range(2))
    if pos is None:
        pos = torch.cat([torch.sort(torch.randint(0, t, (n,), generator=g, device=DEV))[0].int() for t, n in zip(T, sel)])
    shift = torch.zeros(len(T), dtype=torch.int32, device=DEV) if pos0 is None else torch.tensor(pos0, dtype=torch.int32, device=DEV)
    for b in range(len(T)):
        pos[os_[b]:os_[b + 1]] += shift[b]
    o = torch.full((sum(sel), H, 128), float("nan"), device=DEV, dtype=BF)
    lse = torch.full((sum(sel), H), float("nan"), device=DEV)
    desc = qb.make_desc(inputs.LayerShape(2048, H, Hkv, 128, 10000.0, "bf16"))
    qb.qcf_recompute_attn(desc, len(T), q, pos, i64(os_), sum(sel), k, v, i64(oc), sum(T),
                          None if pos0 is None else shift, o, lse)
    for b in range(len(T)):
        rows, ctx = slice(os_[b], os_[b + 1]), slice(oc[b], oc[b + 1])
        seen = torch.arange(T[b], device=DEV)[None] <= (pos[rows] - shift[b])[:, None]
        for h in range(0, H, max(1, H // 16)):                     # (every head of the first groups, then a sample)
            kh, vh = k[ctx, h // (H // Hkv)].double(), v[ctx, h // (H // Hkv)].double()
            s = (q[rows, h].double() @ kh.t() / math.sqrt(128.0)).masked_fill(~seen, -math.inf)
            p = torch.softmax(s, -1).nan_to_num(0.0)
            ref, mass = p @ vh, p @ vh.abs()
            err = (o[rows, h].double() - ref).abs()
            assert bool((err <= 1.02 * 2.0 ** -8 * (mass + ref.abs()) + 1e-6).all()), f"request {b} head {h}: {float(err.max())}"
            ref_lse = torch.logsumexp(s, -1)
            ok = seen.any(-1)
            assert bool(((lse[rows, h].double() - ref_lse).abs()[ok] <= 3e-6 * (1 + ref_lse[ok].abs())).all())
            assert bool((lse[rows, h][~ok] == -math.inf).all()) and bool((o[rows, h][~ok] == 0).all())
    return o, lse


def _assert_wide(H, Hkv, T, sel):
    """The launch has 256 rows to a workgroup; one that is split says so by its workspace."""
    rows, blocks, segments = host_rules.attention(H, Hkv, 128, T, sel)
    assert rows == host_rules.WIDE
    desc = qb.make_desc(inputs.LayerShape(2048, H, Hkv, 128, 10000.0, "bf16"))
    assert qb.qcf_recompute_attn_workspace_bytes(desc, len(T), sum(sel), sum(T)) == (
        host_rules.wide_workspace(Hkv, blocks, segments) if segments > 1 else 0)
    return segments


@pytest.mark.parametrize("H,Hkv,T,sel", [
    (32, 8, 8192, 2457),       # split, four heads to a group
    (64, 8, 8200, 1500),       # split, eight heads, last tile of eight tokens
    (8, 8, 12351, 6100),       # split, one head to a group, last tile one token short
    (128, 32, 3201, 1473),     # whole blocks, one token in the last tile, one row in the last block
    (32, 32, 3300, 5889),
])
def test_one_request(H, Hkv, T, sel):
    say(f"wide attention H={H}/{Hkv} T={T} rows={sel}")
    assert (_assert_wide(H, Hkv, [T], [sel]) > 1) == (Hkv == 8)      # (the others: whole blocks)
    a = _case(80, H, Hkv, [T], [sel])
    b = _case(80, H, Hkv, [T], [sel])
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("q_std", [0.02, 8.0, 60.0], ids=["flat", "sharp", "one-hot"])
def test_logit_range(q_std):
    say(f"wide attention, logits of spread {q_std}")
    _assert_wide(64, 8, [8192], [1229])
    _case(81, 64, 8, [8192], [1229], q_std=q_std)


@pytest.mark.parametrize("H,Hkv,T,sel", [
    (256, 64, [1, 63, 64, 65, 1000, 130, 5, 80000], [1, 64, 64, 128, 400, 0, 200, 3200]),       # one long request among them
    (128, 64, [1, 63, 64, 65, 1000, 130, 5, 400], [1, 64, 64, 128, 700, 0, 200, 130])], ids=["256 rows", "128 rows"])
def test_requests_of_all_lengths(H, Hkv, T, sel):
    """Rows that see nothing, one token, whole tiles; requests without rows or shorter than a tile."""
    say(f"ragged batch of up to {max(T)} tokens")
    if H == 256:
        _assert_wide(H, Hkv, T, sel)
    pos = torch.cat([torch.linspace(0, t - 1, n, device=DEV).int() for t, n in zip(T, sel)])
    _case(82, H, Hkv, T, sel, pos=pos)
    pos = torch.cat([torch.linspace(-3, t + 40, n, device=DEV).int() for t, n in zip(T, sel)])
    _case(83, H, Hkv, T, sel, pos=pos, pos0=[0, 7, 100, 1000, 64, 3, 0, 12345])
