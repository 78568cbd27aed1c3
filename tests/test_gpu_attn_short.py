"""Short attention launches of one request: segments of 2 to 8 key tiles with float partial outputs."""
import pytest

import host_rules
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
