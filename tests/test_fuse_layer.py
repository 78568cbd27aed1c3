"""The layer in one call (qcf_fuse.h): the struct that crosses the boundary, and the bits of the five calls."""
import os
import re
import subprocess

import numpy as np
import pytest
import torch

from oracle import qcf_oracle as orc
from paper_2604_08585_amd import binding as qb
from paper_2604_08585_amd import inputs, pipeline

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_struct_is_packed_as_the_header_lays_it_out(tmp_path):
    text = open(os.path.join(ROOT, "include", "qcf_fuse.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    assert sorted(set(re.findall(r"\b(qcf_[a-z_]+)\s*\(", text))) == qb.FUSE_EXPORTS
    assert hasattr(qb.load_library(), qb.FUSE_EXPORTS[0])
    src = tmp_path / "size.c"
    src.write_text('#include <stdio.h>\n#include <stddef.h>\n#include "qcf_fuse.h"\nint main(void) { typedef qcf_layer_buffers B; '
                   'printf("%zu %zu %zu %zu", sizeof(B), offsetof(B, chunks_dev), offsetof(B, rerope_ws), offsetof(B, rerope_ws_bytes)); }')
    subprocess.run(["gcc", "-I" + os.path.join(ROOT, "include"), str(src), "-o", str(tmp_path / "size")], check=True)
    got = [int(v) for v in subprocess.run([str(tmp_path / "size")], capture_output=True, text=True, check=True).stdout.split()]
    assert got == [qb._LAYER_BUFFERS.size, 32, 32 + 18 * 8, 32 + 23 * 8]


def test_bad_arguments_are_those_of_the_calls():
    desc = qb.make_desc(inputs.LayerShape(256, 4, 2, 64, 10000.0, "f32"))
    lib = qb.load_library()
    import ctypes as C
    assert lib.qcf_fuse_layer(C.byref(desc), None, 1, None) == 1
    args = [1, 1, 8, 0, 4] + [0x1000] * 18 + [0] * 5 + [0] * 5
    args[5 + 7] = 0                                    # k_fused
    assert lib.qcf_fuse_layer(C.byref(desc), qb._LAYER_BUFFERS.pack(*args), 1, None) == 1 and b"k_fused" in lib.qcf_last_error()
    args[5 + 7] = 0x1000
    assert lib.qcf_fuse_layer(C.byref(desc), qb._LAYER_BUFFERS.pack(*args), 1, None) == 3      # no workspace


OUTS = ("k_fused", "v_fused", "score", "sel_idx", "sel_row", "sel_pos", "q_sel", "k_sel", "v_sel", "o_sel", "lse")


@pytest.mark.gpu
@pytest.mark.parametrize("cfg,scale,ratio,critical", [
    (0, 1, 0.15, True), (0, 1, 0.15, False),          # float32, heads of 64
    (2, 1 / 8, 0.15, True), (2, 1 / 8, 0.15, False),  # sixteen ragged chunks
    (2, 1 / 8, 0.0, True),                            # nothing selected
    (1, 1 / 8, 1.0, True), (4, 1 / 64, 0.15, True)])  # everything; a batch
@pytest.mark.parametrize("workspaces", [True, False])
def test_same_bits_as_the_calls_one_after_the_other(cfg, scale, ratio, critical, workspaces):
    print(f"layer in one call cfg={cfg} ratio={ratio} critical={critical}", flush=True)
    L = pipeline.upload(inputs.make_config(cfg, orc.PlantOps(), scale=scale) if cfg else inputs.make_config(cfg, orc.PlantOps()),
                        torch.device("cuda:0"), ratio=ratio)
    if not workspaces:
        L.ws_rerope = L.ws_score = L.ws_select = L.ws_qkv = L.ws_attn = None

    def outputs(run):
        for name in OUTS:
            if critical or name not in ("sel_idx", "sel_row", "sel_pos"):
                getattr(L, name).fill_(1)
        run()
        torch.cuda.synchronize()
        return [getattr(L, name).clone() for name in OUTS]

    def calls():
        for name, fn in pipeline.FUSED_STEPS:
            if critical or name not in ("score", "select"):
                fn(L)

    if not critical:
        pipeline.enqueue_layer(L, fused=False)         # fixes a selection
    want = outputs(calls)
    for _ in range(2):
        for name, a, b in zip(OUTS, outputs(lambda: pipeline.enqueue_layer(L, critical)), want):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), name
