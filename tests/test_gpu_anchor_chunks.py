"""Anchor extraction in one call against key norm, Top-N and gather one after the other, bit for bit: chunks in groups of 448,
empty ones, chunks of every length class, ties, and both sides of the size up to which a workgroup copies its own rows."""
import numpy as np
import pytest
import torch

from paper_2604_08585_amd import binding as qb
from paper_2604_08585_amd import inputs, pipeline
from gpu_util import DEV, i64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("lens,counts", [
    ([300], [300]),                                           # everything
    ([0, 5, 0, 70, 1], [0, 2, 0, 7, 1]),                      # empty chunks
    ([33] * 448, [3] * 448),                                  # one full group
    ([20, 40] * 448 + [9], [1, 2] * 448 + [9]),               # one chunk in the third group
    ([700] * 3, [64, 5, 64]), ([700] * 3, [65, 5, 64]),       # the largest copy of a workgroup (bf16); one row more
    ([1025, 4000, 100], [40, 64, 5]), ([9000, 20], [64, 1]), ([33000], [100])])      # more keys to a thread; read again
def test_extraction_in_one_call(lens, counts, dtype):
    print(f"anchors in one call {lens[:4]} ({len(lens)}) {counts[:4]} {dtype}", flush=True)
    sh = inputs.LayerShape(4096, 32, 8, 128, 500000.0, dtype)
    desc, dt = qb.make_desc(sh), inputs.torch_dtype(dtype)
    g = torch.Generator(device=DEV).manual_seed(len(lens))
    T, M = sum(lens), sum(counts)
    k, v = (torch.randn((T, 8, 128), generator=g, device=DEV).to(dt) for _ in range(2))
    k[T // 3: T // 3 + 20] = k[0]                             # ties
    row, ak, av = pipeline.extract_anchors(desc, k, v, lens, counts)
    norm = torch.empty(T, device=DEV)
    qb.qcf_key_norm(desc, k, T, norm)
    idx, ref = (torch.empty(M, dtype=torch.int32, device=DEV) for _ in range(2))
    ctx_off, sel_off = (i64(np.concatenate([[0], np.cumsum(x)])) for x in (lens, counts))
    qb.qcf_select(len(lens), norm, ctx_off, T, sel_off, M, None, idx, ref, None)
    rk, rv = (torch.empty((M, 8, 128), dtype=dt, device=DEV) for _ in range(2))
    qb.qcf_gather(desc, k, v, ref, M, T, rk, rv)
    torch.cuda.synchronize()
    assert torch.equal(row, ref) and torch.equal(ak, rk) and torch.equal(av, rv)
    assert torch.equal(ak, k[row.long()]) and torch.equal(av, v[row.long()])


@pytest.mark.parametrize("chunks", [63, 64, 65])              # the arguments of a launch hold 64 chunks, or 448
def test_either_size_of_arguments(chunks):
    test_extraction_in_one_call([0, 33, 7] * (chunks // 3) + [40] * (chunks % 3), [0, 3, 7] * (chunks // 3) + [5] * (chunks % 3), "bf16")
