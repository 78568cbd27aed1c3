"""Host arithmetic of the product's division by rows (csrc/gemm_args.h) and into tiles (csrc/gemm_plan.h), compiled and run on the CPU."""
import os
import subprocess

import pytest

import host_rules

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "gemm_args.h"
using namespace qcf;

// every pattern of outputs that are not wanted (bits: q, k, v, fused cache, gather, residual)
template <int EPI> int check(int64_t rows) {
  static bf16_t buf[1];
  static int32_t idx[1];
  int bad = 0;
  for (int m = 0; m < 64; ++m) {
    QkvArgs a{};
    a.x = buf; a.w = buf; a.M = a.x_rows = rows + 77; a.d_model = 512; a.H = 4; a.Hkv = is_rope(EPI) ? 2 : 0; a.D = 128; a.glu = 320;
    a.q = m & 1 ? nullptr : buf;
    a.k = m & 2 || !is_rope(EPI) ? nullptr : buf;
    a.v = m & 4 || !is_rope(EPI) ? nullptr : buf;
    a.pos = is_rope(EPI) ? idx : nullptr;
    if (!(m & 8)) { a.dst_rows = idx; a.k_fused = buf; a.v_fused = buf; }
    if (!(m & 16)) a.gather = idx;
    if (!(m & 32)) a.residual = buf;
    const QkvArgs b = rows_from<EPI>(a, rows);
    const int64_t qc = EPI == kGlu ? 320 : 512;
    bad += b.q != (a.q ? a.q + rows * qc : nullptr);
    bad += b.k != (a.k ? a.k + rows * 256 : nullptr);
    bad += b.v != (a.v ? a.v + rows * 256 : nullptr);
    bad += b.residual != (a.residual ? a.residual + rows * qc : nullptr);
    bad += b.dst_rows != (a.dst_rows ? a.dst_rows + rows : nullptr);
    bad += b.pos != (a.pos ? a.pos + rows : nullptr);
    bad += b.gather != (a.gather ? a.gather + rows : nullptr);
    bad += a.gather ? b.x != a.x || b.x_rows != a.x_rows : b.x != a.x + rows * 512 || b.x_rows != 77;
    bad += b.k_fused != a.k_fused || b.v_fused != a.v_fused || b.w != a.w || b.M != 77;
  }
  return bad;
}

int main() {
  int bad = 0;
  const int64_t cuts[] = {256, 1280, 4864};
  for (int64_t rows : cuts) {
    bad += check<kRopeHalf128>(rows) + check<kRopeHalf64>(rows) + check<kRopeInter>(rows);
    bad += check<kPlain>(rows) + check<kAdd>(rows) + check<kGlu>(rows);
  }
  std::printf("%d\n", bad);
  return bad != 0;
}
"""


def test_a_null_output_stays_null_when_rows_are_cut_off(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I" + os.path.join(ROOT, "paper_2604_08585_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("N,rows,height", [
    (3584, 570, 128), (3584, 615, 96), (3584, 512, 64), (4608, 400, 96), (4608, 384, 64), (4608, 600, 128), (4608, 1344, 224), (4608, 1345, 256),
    (1152, 2305, 128), (3200, 1865, 256), (3200, 1536, 192)])
def test_tiles_fit_a_round_on_every_xcd(N, rows, height):
    """Column blocks, or row tiles, that are no multiple of the eight XCDs: the one that has most of them has a round's workgroups."""
    assert host_rules.tile_rows(rows, N, 4096) == height
    for m in range(65, 3000, 7):
        if host_rules.tile_rows(m, N, 4096) in (64, 96, 160, 192, 224):
            assert host_rules.busiest_xcd(m, N, 4096) <= 32, m


def test_the_least_height_that_fits_is_taken():
    for rows, N, K in ((2000, 1024, 2816), (615, 3072, 2048), (900, 2048, 1536), (320, 6144, 4096), (200, 1024, 1216)):
        assert host_rules.tile_rows(rows, N, K) == 64, (rows, N, K)
    assert host_rules.tile_rows(321, 6144, 4096) == host_rules.tile_rows(350, 6144, 64) == 96


def test_short_contractions_take_tiles_of_96_rows():
    for rows, N, K in ((100, 512, 256), (1000, 512, 256), (1000, 2048, 512), (300, 6144, 1024), (1229, 1024, 1024), (300, 6144, 64)):
        assert host_rules.tile_rows(rows, N, K) == 96, (rows, N, K)


@pytest.mark.parametrize("N,K,rows,height", [
    (4096, 4096, 560, 128), (3584, 4096, 560, 128), (4608, 4096, 560, 128), (4096, 4096, 615, 96), (3072, 2048, 900, 128),
    (3072, 2048, 700, 96), (1024, 2816, 2200, 128), (1024, 2816, 2458, 128), (1024, 2816, 1800, 64), (6144, 4096, 450, 96),
    (8192, 8192, 350, 96), (2048, 6144, 1400, 96), (512, 256, 160, 128), (512, 256, 220, 96)])
def test_a_thin_last_tile_of_128_rows_is_kept(N, K, rows, height):
    """Where tiles of 128 rows fit a round as well, the choice goes by how full the last tile of either height is."""
    assert host_rules.tile_rows(rows, N, K) == height
