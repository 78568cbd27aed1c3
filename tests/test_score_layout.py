"""Workspaces of the scoring: what its launches lay out (csrc/score_layout.h) against what the library reports, on the CPU, and
a batch of more requests than tokens into a workspace of exactly that size."""
import ctypes as C
import os
import subprocess

import pytest
import torch

from paper_2604_08585_amd import binding as qb
from paper_2604_08585_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "score_layout.h"
namespace qcf { int compute_unit_count() { return 256; } }           // (as the library without a device)
using namespace qcf::scoring;

typedef size_t (*One)(const qcf_layer_desc*, int32_t, int64_t, int64_t);
typedef size_t (*Several)(const qcf_layer_desc*, int32_t, int32_t, int64_t, int64_t);

// bytes that the launch of one layer lays out
static size_t one_layer(const qcf_layer_desc& L, int32_t B, int64_t R, int64_t T) {
  if (use_fused(L, B, R, T)) return fused_ws(L, B, T).total;
  if (use_two_pass(L, B, R, T)) return pass_ws(L, 1, B, R, T).total;
  return generic_ws(L, R, T);
}

extern "C" long sweep(const qcf_layer_desc* L, const long* batches, int n_batches, One one, Several several) {
  long bad = 0;
  const long extra[] = {1, 2, 3, 40, 255, 256, 257, 1000, 4096, 6001, 32768, 500000, 1 << 20};
  for (int i = 0; i < n_batches; ++i) {
    const int32_t B = (int32_t)batches[i];
    for (long T : extra)
      for (int64_t R : {1, 16, 500}) {
        const size_t a = one_layer(*L, B, R, T), have = one(L, B, R, T);
        if (a > have && bad++ < 5) std::printf("d=%d B=%d T=%ld R=%ld: %zu > %zu\n", L->head_dim, B, T, (long)R, a, have);
        if (use_two_pass(*L, B, R, T)) {
          const PassWs w = pass_ws(*L, 1, B, R, T);
          // the units of all requests find a place: as many tiles as there can be in as few requests, and spread evenly
          const int64_t full = std::min<int64_t>(B, T);              // requests that are not empty
          int64_t units = 0, left = T;
          for (int64_t b = 0; b < full; ++b) {
            const int64_t t = left / (full - b), nt = (t + kTokPerWg - 1) / kTokPerWg;
            units += (nt + w.unit_tiles - 1) / w.unit_tiles;
            left -= t;
          }
          const int64_t nt = (T - (full - 1) + kTokPerWg - 1) / kTokPerWg;
          bad += units > w.n_units || full - 1 + (nt + w.unit_tiles - 1) / w.unit_tiles > w.n_units;
        }
        for (int n = 1; n <= 33; n += n < 4 ? 1 : 13) {              // 1, 2, 3, 4, 17, 30
          const int at_once = layers_at_once(*L, n, B, R, T), rest = n % at_once;
          size_t need = 0;
          if (at_once == 1 || rest == 1) need = a;
          if (at_once > 1) need = std::max(need, pass_ws(*L, at_once, B, R, T).total);
          if (rest > 1) need = std::max(need, pass_ws(*L, rest, B, R, T).total);
          bad += need > several(L, n, B, R, T);
        }
      }
  }
  return bad;
}
"""


@pytest.mark.parametrize("H,Hkv,D", [(32, 8, 128), (64, 8, 128), (32, 8, 64), (8, 8, 128), (4, 1, 64)])
def test_launches_stay_inside_the_reported_workspace(tmp_path, H, Hkv, D):
    src, so = tmp_path / "t.cpp", tmp_path / "t.so"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2604_08585_amd", "csrc"), str(src), "-o", str(so)], check=True)
    lib = qb.load_library()
    sweep = C.CDLL(str(so)).sweep
    sweep.restype = C.c_long
    batches = list(range(1, 20)) + list(range(20, 700, 7)) + list(range(700, 65535, 1500)) + [256, 257, 258, 259, 260, 300, 65534, 65535]
    desc = qb.make_desc(inputs.LayerShape(2048, H, Hkv, D, 10000.0, "bf16"))
    address = lambda f: C.cast(f, C.c_void_p)
    assert sweep(C.byref(desc), (C.c_long * len(batches))(*batches), len(batches), address(lib.qcf_score_workspace_bytes),
                 address(lib.qcf_score_layers_workspace_bytes)) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("H,Hkv,D", [(32, 8, 128), (32, 8, 64)])
def test_more_requests_than_tokens(H, Hkv, D):
    """300 requests, all but three empty, against float64; the bytes behind the workspace stay as they were."""
    from test_gpu_score_units import REL, _inputs, _reference
    from gpu_util import DEV, i64
    print(f"scores of 300 requests, three not empty, D={D}", flush=True)
    T, R = [0] * 300, [0] * 300
    T[0], T[150], T[299] = 5, 34, 1
    R[0], R[7], R[150], R[299] = 3, 2, 60, 1
    q, k, oq, ok, _ = _inputs(62, 2, H, Hkv, D, T, R)
    desc = qb.make_desc(inputs.LayerShape(2048, H, Hkv, D, 10000.0, "bf16"))
    ref = [_reference(q[l], k[l], oq, ok) for l in range(2)]

    def guarded(need):
        ws = torch.full((need + (1 << 21),), 0x5a, dtype=torch.uint8, device=DEV)
        return ws, ws[:need]

    whole, ws = guarded(qb.qcf_score_workspace_bytes(desc, 300, sum(R), sum(T)))
    score = torch.full((sum(T),), float("nan"), device=DEV)
    qb.qcf_score(desc, 300, q[0], i64(oq), sum(R), k[0], i64(ok), sum(T), None, score, ws)
    assert float((score.double() - ref[0]).norm() / ref[0].norm()) < REL
    assert bool((whole[ws.numel():] == 0x5a).all())
    need = qb.load_library().qcf_score_layers_workspace_bytes(C.byref(desc), 2, 300, sum(R), sum(T))
    whole, ws = guarded(need)
    qb.qcf_score_layers(desc, 300, q, i64(oq), sum(R), k, i64(ok), sum(T), None, [1.0, 0.5], score, ws)
    both = ref[0] + 0.5 * ref[1]
    assert float((score.double() - both).norm() / both.norm()) < REL
    assert bool((whole[ws.numel():] == 0x5a).all())
