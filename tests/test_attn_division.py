"""Which attention launches take 256 rows to a workgroup (csrc/attn_layout.h), on the CPU."""
import pytest

import host_rules


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
