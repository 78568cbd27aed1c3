"""The library's host rules, compiled from their headers for the tests (csrc/attn_layout.h, gemm_plan.h and score_layout.h; 256
compute units)."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

from paper_2604_08585_amd import binding as qb
from paper_2604_08585_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WIDE = 256

PROGRAM = r"""
#include "attn_layout.h"
#include "gemm_plan.h"
#include "score_layout.h"
namespace qcf { int compute_unit_count() { return 256; } }
extern "C" void division(const qcf_layer_desc* L, int B, long long rows, long long tokens, long long* out) {
  const qcf::attn::Division d = qcf::attn::divide(*L, B, rows, tokens);
  out[0] = d.rows; out[1] = d.n_row_blocks; out[2] = d.split.n_seg_max;
}
// least and full workspace, and what the division takes that a workspace of `have` bytes gives
extern "C" void attention_workspace(const qcf_layer_desc* L, int B, long long rows, long long tokens, long long have, long long* out) {
  using namespace qcf::attn;
  out[0] = least_workspace(*L, B, rows, tokens);
  out[1] = full_workspace(*L, B, rows, tokens);
  const Division d = divide(*L, B, rows, tokens, have);
  out[2] = workspace_of(*L, d); out[3] = d.split.n_seg_max; out[4] = d.split.part_f32;
}
extern "C" int takes_rerope(const qcf_layer_desc* L, int B, int n_chunks, long long probes, long long tokens) {
  return qcf::scoring::takes_rerope(*L, B, n_chunks, probes, tokens);
}
extern "C" int pass1_takes_rerope(const qcf_layer_desc* L, int B, int n_chunks, long long probes, long long tokens) {
  return qcf::scoring::pass1_takes_rerope(*L, B, n_chunks, probes, tokens);
}
extern "C" int pass1_rerotates(const qcf_layer_desc* L, int unit_tiles, int n_layers, int limit) {
  return qcf::scoring::pass1_rerotates(*L, unit_tiles, n_layers, limit);
}
extern "C" int unit_tiles(const qcf_layer_desc* L, int B, long long probes, long long tokens) {
  return qcf::scoring::pass_ws(*L, 1, B, probes, tokens).unit_tiles;
}
extern "C" int sums_in_selection(const qcf_layer_desc* L, int B, long long probes, long long tokens) {
  return qcf::scoring::sums_in_selection(*L, B, probes, tokens);
}
extern "C" int tile_rows(long long rows, int columns, int contraction, long long workspace) {
  using namespace qcf::gemm;
  const ProductPlan p = plan_product(rows, columns / kBN, contraction / kBK, true, workspace);
  return p.blocks != 0 || p.rest.splits > 1 ? 0 : rows_of(p.rest.kind);
}
// ranges that the contraction of a projection in one launch of tiles of 64 to 256 rows is cut into (-1: in other launches), with
// the cache re-rotated beside it and without
extern "C" int ranges(const qcf_layer_desc* L, long long rows, long long workspace, int beside) {
  using namespace qcf::gemm;
  const ProductPlan p = plan_product(rows, (L->n_q_heads + 2 * L->n_kv_heads) * L->head_dim / kBN, L->d_model / kBK, true, workspace, !beside);
  return p.blocks == 0 ? p.rest.splits : -1;
}
// workgroups of the product on the XCD that has most of them, by the order of the launch (0: divided, or 256 x 256 tiles)
extern "C" long long busiest_xcd(long long rows, int columns, int contraction, long long workspace) {
  using namespace qcf::gemm;
  const ProductPlan p = plan_product(rows, columns / kBN, contraction / kBK, true, workspace);
  if (p.blocks != 0 || p.rest.splits > 1) return 0;
  const int units = columns / kBN, mt = (int)((rows + rows_of(p.rest.kind) - 1) / rows_of(p.rest.kind));
  long long n[8] = {0};
  for (int m = 0; m < mt; ++m)
    for (int u = 0; u < units; ++u) ++n[(mt >= kRowsOverXcds ? m : u) % 8];
  return *std::max_element(n, n + 8);
}
extern "C" long long side_rows(const qcf_layer_desc* L, long long rows, int n_chunks, long long tokens, long long workspace) {
  return qcf::gemm::side_rows(*L, rows, n_chunks, tokens, workspace).all;
}
"""


@functools.lru_cache(None)
def _library():
    folder = tempfile.mkdtemp()
    src, so = os.path.join(folder, "rules.cpp"), os.path.join(folder, "rules.so")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2604_08585_amd", "csrc"), src, "-o", so], check=True)
    return C.CDLL(so)


def attention(H, Hkv, D, T, sel):
    """Rows of a workgroup, row blocks (upper bound) and key segments that the attention of these requests is divided into."""
    desc = qb.make_desc(inputs.LayerShape(2048, H, Hkv, D, 10000.0, "bf16"))
    out = (C.c_longlong * 3)()
    _library().division(C.byref(desc), len(T), C.c_longlong(sum(sel)), C.c_longlong(sum(T)), out)
    return tuple(out)


def attention_workspace(H, Hkv, D, T, sel, have=0):
    """Bytes of workspace without which the attention of these requests is refused (heads of 128), bytes that are reported, and
    of the division with `have` bytes of it: its own bytes, key segments, whether they are short ones."""
    desc = qb.make_desc(inputs.LayerShape(2048, H, Hkv, D, 10000.0, "bf16"))
    out = (C.c_longlong * 5)()
    _library().attention_workspace(C.byref(desc), len(T), C.c_longlong(sum(sel)), C.c_longlong(sum(T)), C.c_longlong(have), out)
    return tuple(out)


def rerotates_in_scoring(L):
    """Whether a scored pipeline.DeviceLayer is re-rotated by its scoring kernel (csrc/score_layout.h)."""
    return bool(_library().takes_rerope(C.byref(L.desc), L.B, L.n_chunks, C.c_longlong(L.total_probe), C.c_longlong(L.total_ctx)))


def rerotates_in_pass1(L):
    """Whether a scored pipeline.DeviceLayer with heads of 64 is re-rotated by the first pass of its scoring (csrc/score_layout.h)."""
    return bool(_library().pass1_takes_rerope(C.byref(L.desc), L.B, L.n_chunks, C.c_longlong(L.total_probe), C.c_longlong(L.total_ctx)))


def pass1_rerotates(desc, unit_tiles, layers, limit):
    """Whether the first scoring pass has a kernel that re-rotates for launches of this form, whoever asks for it (csrc/score_layout.h)."""
    return bool(_library().pass1_rerotates(C.byref(desc), unit_tiles, layers, int(limit)))


def unit_tiles(desc, B, probes, tokens):
    """Tiles to a unit of the two scoring passes over one layer."""
    return _library().unit_tiles(C.byref(desc), B, C.c_longlong(probes), C.c_longlong(tokens))


def sums_in_selection(L):
    """What the selection adds up of a pipeline.DeviceLayer's scoring (csrc/score_layout.h): 0 nothing, 1 column sums of the heads, 2
    probability rows."""
    return _library().sums_in_selection(C.byref(L.desc), L.B, C.c_longlong(L.total_probe), C.c_longlong(L.total_ctx))


def tile_rows(M, N, K, workspace=0):
    """Rows of a tile of a bf16 product in one undivided launch (csrc/gemm_plan.h); 0: divided, or 256 x 256 tiles."""
    return _library().tile_rows(C.c_longlong(M), N, K, C.c_longlong(workspace))


def busiest_xcd(M, N, K, workspace=0):
    """Workgroups on the XCD that has most of them, of a bf16 product in one undivided launch; 0: divided, or 256 x 256 tiles."""
    f = _library().busiest_xcd
    f.restype = C.c_longlong
    return f(C.c_longlong(M), N, K, C.c_longlong(workspace))


def ranges_of_projection(desc, rows, tokens, workspace):
    """Ranges that the contraction of a projection of `rows` rows is cut into where the cache of `tokens` rows is re-rotated beside it,
    and where it is not; None: it is not re-rotated beside it."""
    lib, desc, rows, ws = _library(), C.byref(desc), C.c_longlong(rows), C.c_longlong(workspace)
    lib.side_rows.restype = C.c_longlong
    if lib.side_rows(desc, rows, 8, C.c_longlong(tokens), ws) <= 0:
        return None
    return lib.ranges(desc, rows, ws, 1), lib.ranges(desc, rows, ws, 0)


def rows_beside_projection(L):
    """Rows of a layer that is not scored that are re-rotated beside its projection (csrc/gemm_plan.h)."""
    f = _library().side_rows
    f.restype = C.c_longlong
    have = qb.qcf_recompute_qkv_workspace_bytes(L.desc, L.total_sel)
    return f(C.byref(L.desc), C.c_longlong(L.total_sel), L.n_chunks, C.c_longlong(L.total_ctx), C.c_longlong(have))


def wide_workspace(Hkv, blocks, segments):
    """Bytes of a split launch of wide workgroups: partial outputs and log-sum-exps in float32, the list of units, the lengths
    of the row blocks."""
    up = lambda n: (n + 255) // 256 * 256
    rows = blocks * Hkv * segments * WIDE
    return up(rows * 128 * 4) + up(rows * 4) + up((blocks * segments + 1) * 4) + up(blocks * 4)
