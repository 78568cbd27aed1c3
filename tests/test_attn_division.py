"""Which attention launches take 256 rows to a workgroup (csrc/attn_layout.h), on the CPU."""
import pytest

import host_rules
from paper_2604_08585_amd import binding as qb
from paper_2604_08585_amd import inputs


@pytest.mark.parametrize("H,Hkv", [(32, 8), (64, 8)])
@pytest.mark.parametrize("B,T,rows", [
    (130, 100, 5), (130, 8000, 5), (200, 300, 10), (256, 256, 39), (1000, 1, 1),      # blocks that are mostly empty
    (64, 1000, 150), (128, 512, 77), (40, 1500, 225),                                 # short contexts
    (12, 4096, 614), (2, 8192, 410)])                                                 # little work to a compute unit
def test_batches_of_short_or_few_rows_keep_128(H, Hkv, B, T, rows):
    assert host_rules.attention(H, Hkv, 128, [T] * B, [rows] * B)[0] == 128


@pytest.mark.parametrize("H,Hkv,T,rows", [
    (32, 8, [12288] * 17, [1843] * 17), (64, 8, [16384] * 4, [2457] * 4),
    (32, 8, [2048 * n for n in (1, 2, 3, 4, 5, 6, 7, 8)] * 2, [307 * n for n in (1, 2, 3, 4, 5, 6, 7, 8)] * 2)])
def test_long_batches_take_256(H, Hkv, T, rows):
    assert host_rules.attention(H, Hkv, 128, T, rows)[0] == host_rules.WIDE


def test_one_request_whose_blocks_are_not_filled():
    for H, Hkv, T, rows in [(32, 32, 23078, 876), (32, 32, 8509, 2572), (64, 8, 24576, 491), (256, 256, 3100, 257)]:
        assert host_rules.attention(H, Hkv, 128, [T], [rows])[0] == 128


def test_one_request():
    assert host_rules.attention(32, 8, 128, [8192], [1229])[0] == 128
    assert host_rules.attention(32, 8, 128, [8192], [2457])[0] == host_rules.WIDE
    assert host_rules.attention(64, 8, 128, [32768], [4915])[0] == host_rules.WIDE
    assert host_rules.attention(32, 8, 64, [32768], [9830])[0] == 128


@pytest.mark.parametrize("H,Hkv,D", [(32, 8, 128), (64, 8, 128), (16, 16, 128), (32, 8, 64)])
def test_workspace_that_is_reported_and_the_least_one(H, Hkv, D):
    """Short segments are taken where the workspace holds them, and never asked for: any size from the least one on gets a division
    that fits, the reported one gets the division that the rule wants."""
    desc = qb.make_desc(inputs.LayerShape(2048, H, Hkv, D, 10000.0, "bf16"))
    short = 0
    for T in (64, 200, 512, 731, 1000, 2048, 3000, 6001, 8192):
        for rows in sorted({1, 30, 77, 110, 300, 450, 614, int(0.15 * T) + 1, T}):
            least, full, *_ = host_rules.attention_workspace(H, Hkv, D, [T], [rows])
            assert least <= full == qb.qcf_recompute_attn_workspace_bytes(desc, 1, rows, T)
            for have in sorted({max(least - 1, 0), least, (least + full) // 2, full - 1, full, 2 * full}):
                _, _, takes, segments, is_short = host_rules.attention_workspace(H, Hkv, D, [T], [rows], have)
                assert takes <= max(least, have) and (takes == least or is_short)
                if have >= full:
                    assert segments == host_rules.attention(H, Hkv, D, [T], [rows])[2]
                    short += is_short
    assert short > 0


def test_least_workspace_is_that_of_the_plain_division():
    """32 query and 8 KV heads of 128: nothing where blocks stay whole, bf16 partial outputs and no more where they do not."""
    least = lambda T, rows: host_rules.attention_workspace(32, 8, 128, [T], [rows])[0]
    up = lambda n: (n + 255) // 256 * 256
    assert least(512, 77) == least(512, 110) == 0
    for T, rows, segments in [(731, 110, 2), (3000, 77, 6), (3000, 110, 6)]:
        units = ((rows + 31) // 32 + 1) * segments
        assert least(T, rows) == up(units * 8 * 128 * 128 * 2) + up(units * 8 * 128 * 4) + up((units + 1) * 4) + up(units // segments * 4)
