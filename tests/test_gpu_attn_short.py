"""Short attention launches of one request: segments of 2 to 8 key tiles with float partial outputs."""
import pytest

import host_rules
from paper_2604_08585_amd import binding as qb
from paper_2604_08585_amd import inputs
import test_gpu_attn_order as order

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["end", "two places", "out of order", "none visible"])
@pytest.mark.parametrize("H,Hkv,D,T,n,segments", [
    (32, 8, 128, 513, 1, 5),        # one row, one token in the last of nine tiles
    (32, 8, 64, 449, 33, 4),        # one row in the second row block
    (16, 16, 128, 640, 129, 5),     # one head to a group
    (64, 8, 128, 731, 31, 6),       # eight: a block that lacks one row
    (32, 8, 128, 731, 110, 4),
    (32, 8, 128, 1000, 150, 4),
    (32, 8, 64, 2047, 100, 8),
    (32, 8, 128, 448, 40, 1)])      # whole: the merge would cost more
def test_short_segments(H, Hkv, D, T, n, segments, kind):
    assert host_rules.attention(H, Hkv, D, [T], [n])[2] == segments
    order.test_order_of_units(H, Hkv, D, T, n, kind)


@pytest.mark.parametrize("H,Hkv,D,T,n", [
    (32, 8, 128, 512, 77),          # none
    (32, 8, 128, 731, 110), (32, 8, 128, 731, 300), (32, 8, 128, 2048, 100), (64, 8, 128, 731, 31),
    (32, 8, 64, 731, 110)])         # (optional, but taken)
def test_least_workspace(H, Hkv, D, T, n, monkeypatch):
    """A caller whose workspace holds the division of longer launches only, or who has none where that takes none."""
    least, full, *_ = host_rules.attention_workspace(H, Hkv, D, [T], [n])
    assert least < full == qb.qcf_recompute_attn_workspace_bytes(qb.make_desc(inputs.LayerShape(2048, H, Hkv, D, 10000.0, "bf16")), 1, n, T)
    assert not host_rules.attention_workspace(H, Hkv, D, [T], [n], least)[4]
    monkeypatch.setattr(qb, "qcf_recompute_attn_workspace_bytes", lambda *a: least)
    order.test_order_of_units(H, Hkv, D, T, n, "spread")
    order.test_order_of_units(H, Hkv, D, T, n, "none visible")
    if D == 128 and least:
        monkeypatch.setattr(qb, "qcf_recompute_attn_workspace_bytes", lambda *a: least - 1)
        with pytest.raises(qb.QcfError, match="TOO_SMALL"):
            order.test_order_of_units(H, Hkv, D, T, n, "spread")
