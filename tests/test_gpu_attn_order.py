"""Split attention of one request: every workgroup works out the order of the units from the positions.  Rows gathered in one
place, rows out of order, rows that see nothing, and the sizes at which the order comes from a launch of its own."""
import math

import pytest
import torch

from paper_2604_08585_amd import binding as qb
from paper_2604_08585_amd import inputs
from gpu_util import DEV, i64

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


def _positions(kind, T, n, g):
    if kind == "end":
        return torch.arange(T - n, T, device=DEV, dtype=torch.int32)
    if kind == "two places":
        return torch.cat([torch.arange(n // 2, device=DEV), torch.arange(T - n + n // 2, T, device=DEV)]).int()
    pos = torch.randperm(T, generator=g, device=DEV)[:n].int()
    if kind == "none visible":
        pos[: n // 3] = -1
    return pos if kind == "out of order" else torch.sort(pos)[0]


@pytest.mark.parametrize("kind", ["end", "two places", "out of order", "none visible"])
@pytest.mark.parametrize("H,Hkv,D,T,n", [
    (32, 8, 128, 4096, 615),        # 21 row blocks
    (32, 8, 64, 4033, 577),         # one row in the last block with rows, one token in the last tile
    (32, 8, 128, 8192, 1057),
    (64, 8, 128, 6000, 1700),       # 256 rows to a workgroup
    (16, 16, 128, 2048, 1100),      # one head to a group
    (8, 1, 128, 16384, 1000),       # more than 512 units: ordered by a launch
])
def test_order_of_units(H, Hkv, D, T, n, kind):
    """Probabilities, the partial results of 128-row workgroups (heads of 128) and the result are rounded to bf16, each by at
    most 2^-8 of the value: |error| <= 2^-8 (2 sum p |v| + |o|), and a little for the 32-bit sums."""
    print(f"attention units H={H}/{Hkv} D={D} T={T} rows={n} {kind}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(T + n)
    q = torch.randn((n, H, D), generator=g, device=DEV, dtype=BF)
    k, v = (torch.randn((T, Hkv, D), generator=g, device=DEV, dtype=BF) for _ in range(2))
    pos = _positions(kind, T, n, g)
    o = torch.full((n, H, D), float("nan"), device=DEV, dtype=BF)
    lse = torch.full((n, H), float("nan"), device=DEV)
    desc = qb.make_desc(inputs.LayerShape(2048, H, Hkv, D, 10000.0, "bf16"))
    qb.qcf_recompute_attn(desc, 1, q, pos, i64([0, n]), n, k, v, i64([0, T]), T, None, o, lse)
    seen = torch.arange(T, device=DEV)[None] <= pos[:, None]
    for h in range(0, H, max(1, H // 8)):
        kh, vh = k[:, h // (H // Hkv)].double(), v[:, h // (H // Hkv)].double()
        s = (q[:, h].double() @ kh.t() / math.sqrt(D)).masked_fill(~seen, -math.inf)
        p = torch.softmax(s, -1).nan_to_num(0.0)
        ref, mass = p @ vh, p @ vh.abs()
        err = (o[:, h].double() - ref).abs()
        assert bool((err <= 1.02 * 2.0 ** -8 * (2 * mass + ref.abs()) + 1e-6).all()), f"head {h}: {float(err.max())}"
        ok = seen.any(-1)
        ref_lse = torch.logsumexp(s, -1)
        assert bool(((lse[:, h].double() - ref_lse).abs()[ok] <= 3e-6 * (1 + ref_lse[ok].abs())).all())
        assert bool((lse[:, h][~ok] == -math.inf).all()) and bool((o[:, h][~ok] == 0).all())
