"""What the host does around a launch: the stream that a call goes to, the offset tables of the anchor extraction."""
import numpy as np
import pytest
import torch

from paper_2604_08585_amd import binding as qb
from paper_2604_08585_amd import inputs, pipeline
from gpu_util import DEV

pytestmark = pytest.mark.gpu


def test_calls_go_to_the_current_stream():
    torch.zeros(1, device=DEV)
    assert qb._stream() == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert qb._stream() == side.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert qb._stream() == torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("lens,counts", [([7], [7]), ([5, 1, 300], [9, 1, 0]), (np.array([64, 33]), np.array([3, 40])),
                                         ([12, 8], [2, 3, 4])], ids=["one", "clamped", "arrays", "one count too many"])
def test_anchor_offsets(lens, counts):
    print(f"anchors {lens} {counts}", flush=True)
    sh = inputs.LayerShape(512, 8, 2, 64, 10000.0, "f32")
    g = torch.Generator(device=DEV).manual_seed(90)
    k, v = (torch.randn((int(sum(lens)), 2, 64), generator=g, device=DEV) for _ in range(2))
    row, ak, av = pipeline.extract_anchors(qb.make_desc(sh), k, v, lens, counts)
    want, first = [], 0
    for n, c in zip(lens, counts):
        norm = k[first:first + n].double().flatten(1).norm(dim=1)
        want.append(torch.sort(torch.topk(norm, min(int(c), int(n)))[1])[0] + first)
        first += int(n)
    want = torch.cat(want)
    assert torch.equal(row.long(), want) and torch.equal(ak, k[want]) and torch.equal(av, v[want])
