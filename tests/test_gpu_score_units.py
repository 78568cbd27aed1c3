"""Scoring in two passes: units of several tiles, blocks of probe rows, layers that share their launches."""
import ctypes as C
import math

import pytest
import torch

from paper_2604_08585_amd import binding as qb
from paper_2604_08585_amd import inputs, pipeline
from gpu_util import DEV, i64

BF = torch.bfloat16


def say(msg):
    print(msg, flush=True)


def _reference(q, k, offs_q, offs_k, limit=None):
    """Mean over heads and probe rows of the softmax, request by request, in float64."""
    G, out = q.shape[1] // k.shape[1], []
    for b in range(len(offs_q) - 1):
        qb_, kb = q[offs_q[b]:offs_q[b + 1]].double(), k[offs_k[b]:offs_k[b + 1]].double()
        if not len(qb_):
            out.append(torch.zeros(len(kb), dtype=torch.float64, device=q.device))
            continue
        s = qb_.transpose(0, 1) @ kb.repeat_interleave(G, dim=1).permute(1, 2, 0).contiguous() / math.sqrt(q.shape[2])
        if limit is not None:
            lim = limit[offs_q[b]:offs_q[b + 1]].long()
            s.masked_fill_(torch.arange(len(kb), device=q.device)[None, None] >= lim[None, :, None], -math.inf)
        out.append(torch.softmax(s, -1).nan_to_num(0.0).mean((0, 1)))
    return torch.cat(out)


def _inputs(seed, n_layers, H, Hkv, D, T, R):
    g = torch.Generator(device=DEV).manual_seed(seed)
    q = [torch.randn((sum(R), H, D), generator=g, device=DEV, dtype=BF) for _ in range(n_layers)]
    k = [torch.randn((sum(T), Hkv, D), generator=g, device=DEV, dtype=BF) for _ in range(n_layers)]
    off = lambda v: [sum(v[:i]) for i in range(len(v) + 1)]
    return q, k, off(R), off(T), g


# sums of 32-bit exponentials of 32-bit logits: rounding of about 20 operations per term
REL = 3e-6


@pytest.mark.gpu
@pytest.mark.parametrize("limited", [False, True])
@pytest.mark.parametrize("H,Hkv,D,T,R", [
    (32, 8, 128, [20000], [90]),                            # units of several tiles, the last shorter; two row blocks
    (16, 8, 64, [9000, 1, 16384, 257], [3, 5, 0, 41]),      # a request without probe rows, one token, one past a tile
    (32, 8, 128, [256 * 40, 256 * 33 + 64, 5], [80, 81, 1]),       # whole tiles, a quarter of a tile
], ids=["long", "heads64", "batch"])
def test_units_of_several_tiles(H, Hkv, D, T, R, limited):
    say(f"score units H={H}/{Hkv} D={D} T={T} R={R} limited={limited}")
    q, k, oq, ok, g = _inputs(60, 1, H, Hkv, D, T, R)
    lim = torch.randint(0, max(T) + 1, (sum(R),), generator=g, device=DEV, dtype=torch.int32) if limited else None
    if limited:
        lim[0] = 0
    desc = qb.make_desc(inputs.LayerShape(2048, H, Hkv, D, 10000.0, "bf16"))
    score = torch.full((sum(T),), float("nan"), device=DEV)
    qb.qcf_score(desc, len(T), q[0], i64(oq), sum(R), k[0], i64(ok), sum(T), lim, score)
    ref = _reference(q[0], k[0], oq, ok, lim)
    assert float((score.double() - ref).norm() / ref.norm()) < REL
    assert bool(((score.double() - ref).abs() <= 1e-5 * ref + 1e-12).all())


@pytest.mark.gpu
@pytest.mark.parametrize("limited", [False, True])
@pytest.mark.parametrize("H,Hkv,D,T,R", [
    (32, 8, 128, [257], [81]),                              # 324 rows of a group: a second block of four
    (12, 3, 128, [1, 256, 1000], [161, 0, 80]),             # three KV heads; one token, a whole tile
    (8, 8, 64, [255, 2048], [321, 641]),                    # one row past a block, one past two
    (32, 8, 64, [700], [1])], ids=["two blocks", "batch", "heads64", "one row"])
def test_units_of_one_tile(H, Hkv, D, T, R, limited):
    say(f"score units of one tile H={H}/{Hkv} D={D} T={T} R={R} limited={limited}")
    q, k, oq, ok, g = _inputs(63, 1, H, Hkv, D, T, R)
    lim = torch.randint(0, max(T) + 1, (sum(R),), generator=g, device=DEV, dtype=torch.int32) if limited else None
    if limited:
        lim[0], lim[-1] = max(T), 0
    desc = qb.make_desc(inputs.LayerShape(2048, H, Hkv, D, 10000.0, "bf16"))
    score = torch.full((sum(T),), float("nan"), device=DEV)
    qb.qcf_score(desc, len(T), q[0], i64(oq), sum(R), k[0], i64(ok), sum(T), lim, score)
    ref = _reference(q[0], k[0], oq, ok, lim)
    assert bool(((score.double() - ref).abs() <= 1e-5 * ref + 1e-12).all())
    qb.qcf_score_accumulate(desc, len(T), q[0], i64(oq), sum(R), k[0], i64(ok), sum(T), lim, -0.5, 2.0, score)
    assert bool(((score.double() - 1.5 * ref).abs() <= 3e-5 * ref + 1e-12).all())


@pytest.mark.gpu
@pytest.mark.parametrize("n_layers,D,T,R", [
    (2, 128, [1], [1]), (3, 128, [255], [7]), (5, 128, [6001], [48]), (17, 128, [513], [20]),    # 17: a second set of launches
    (33, 128, [40, 700], [2, 9]), (4, 128, [300, 64, 1025], [5, 0, 17]), (3, 64, [400], [12]), (1, 128, [900], [24])])
def test_layers_that_share_their_launches(n_layers, D, T, R):
    say(f"score layers n={n_layers} D={D} T={T} R={R}")
    H, Hkv = 16, 4
    q, k, oq, ok, _ = _inputs(61, n_layers, H, Hkv, D, T, R)
    w = [(-1.0) ** l / (l + 1.0) if n_layers == 5 else 1.0 / (l + 1.0) for l in range(n_layers)]
    desc = qb.make_desc(inputs.LayerShape(2048, H, Hkv, D, 10000.0, "bf16"))
    got = pipeline.score_over_layers(desc, q, k, i64(oq), i64(ok), w)
    one = torch.full((sum(T),), float("nan"), device=DEV)
    for l in range(n_layers):
        qb.qcf_score_accumulate(desc, len(T), q[l], i64(oq), sum(R), k[l], i64(ok), sum(T), None, w[l], float(l > 0), one)
    parts = [x * _reference(q[l], k[l], oq, ok) for l, x in enumerate(w)]
    ref, scale = sum(parts), sum(p.abs() for p in parts)         # (weights of both signs cancel)
    for s in (got, one):
        assert bool(((s.double() - ref).abs() <= 1e-5 * scale + 1e-12).all())
    again = pipeline.score_over_layers(desc, q, k, i64(oq), i64(ok), w)
    assert torch.equal(got, again)


def test_arguments_of_the_call_over_layers():
    lib = qb.load_library()
    fake = 0x1000          # aligned, never dereferenced: validation fails before any launch
    ptrs, w = (C.c_void_p * 2)(fake, fake), (C.c_float * 2)(1.0, 1.0)
    desc = qb.make_desc(inputs.LayerShape(512, 16, 4, 128, 10000.0, "bf16"))
    call = lambda n=2, q=ptrs, k=ptrs, weights=w, ws=fake, have=1 << 30, score=fake: lib.qcf_score_layers(
        C.byref(desc), n, 1, q, fake, 20, k, fake, 512, None, weights, score, ws, have, None)
    need = lib.qcf_score_layers_workspace_bytes(C.byref(desc), 2, 1, 20, 512)
    assert need >= qb.qcf_score_workspace_bytes(desc, 1, 20, 512) > 0
    assert call(n=0) == 1 and call(q=None) == 1 and call(weights=None) == 1 and call(score=None) == 1
    assert call(k=(C.c_void_p * 2)(fake, None)) == 1 and call(k=(C.c_void_p * 2)(fake, fake + 4)) == 1
    assert call(weights=(C.c_float * 2)(1.0, math.inf)) == 1
    assert call(ws=None, have=0) == 3 and call(have=need - 1) == 3
    # many layers do not make the workspace grow without bound
    for T, R in [(512, 20), (6001, 48), (1 << 20, 4096)]:
        one = qb.qcf_score_workspace_bytes(desc, 1, R, T)
        assert lib.qcf_score_layers_workspace_bytes(C.byref(desc), 1000, 1, R, T) <= max(one, 64 << 20)
