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
    _check_anchors(lens, counts, counts)


@pytest.mark.parametrize("given", [lambda c: (v for v in c), lambda c: torch.tensor(c, device=DEV),
                                   lambda c: [torch.tensor(v, device=DEV) for v in c], lambda c: [v + 0.5 for v in c]],
                         ids=["generator", "tensor", "tensors", "fractions"])
def test_anchor_counts_of_any_kind(given):
    print("anchor counts", flush=True)
    _check_anchors([40, 9, 300], given([3, 12, 7]), [3, 12, 7])


def test_counts_for_each_chunk():
    for counts in ([4], [], [4, 4]):
        with pytest.raises(ValueError):
            _check_anchors([40, 9, 300], counts, [4, 4, 4])


def test_weights_of_any_kind():
    sh = inputs.LayerShape(512, 8, 2, 64, 10000.0, "f32")
    g = torch.Generator(device=DEV).manual_seed(91)
    q = [torch.randn((3, 8, 64), generator=g, device=DEV) for _ in range(2)]
    k = [torch.randn((70, 2, 64), generator=g, device=DEV) for _ in range(2)]
    off = [torch.tensor([0, n], dtype=torch.int64, device=DEV) for n in (3, 70)]
    want = pipeline.score_over_layers(qb.make_desc(sh), q, k, *off, [0.25, 0.75])
    for w in ((v for v in (0.25, 0.75)), torch.tensor([0.25, 0.75]), (0.25, 0.75, 9.0)):
        assert torch.equal(pipeline.score_over_layers(qb.make_desc(sh), q, k, *off, w), want)


def _check_anchors(lens, given, counts):
    sh = inputs.LayerShape(512, 8, 2, 64, 10000.0, "f32")
    g = torch.Generator(device=DEV).manual_seed(90)
    k, v = (torch.randn((int(sum(lens)), 2, 64), generator=g, device=DEV) for _ in range(2))
    row, ak, av = pipeline.extract_anchors(qb.make_desc(sh), k, v, lens, given)
    want, first = [], 0
    for n, c in zip(lens, counts):
        norm = k[first:first + n].double().flatten(1).norm(dim=1)
        want.append(torch.sort(torch.topk(norm, min(int(c), int(n)))[1])[0] + first)
        first += int(n)
    want = torch.cat(want)
    assert torch.equal(row.long(), want) and torch.equal(ak, k[want]) and torch.equal(av, v[want])
