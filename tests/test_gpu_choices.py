"""The Bcast of degree-ordered roots takes the copy where its tests say so:
not under capture, and not for units either side of its rule."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2102_13018_amd import inputs
from paper_2102_13018_amd import sf as S

pytestmark = pytest.mark.gpu
R, L = 1_000_003, 2_500_001


@pytest.fixture(scope="module")
def graph():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return inputs.spmv_ghost(seed=90, nroots=R, nleaves=L, zipf_s=1.2, nseg=17)


def copied(sf, dtype, bs, stream=None):
    shape = (lambda n: (n,) if bs == 1 else (n, bs))
    root = torch.zeros(shape(R), dtype=dtype, device="cuda")
    leaf = torch.ones(shape(L), dtype=dtype, device="cuda")
    sf.bcast(root, leaf, stream=stream)
    torch.cuda.synchronize()
    return sf.choices()["last_bcast_copied"]


def test_units(graph):
    sf = S.StarForest(R, graph.iroot, None, graph.ranks).setup()
    assert copied(sf, torch.float64, 1) == 1 and copied(sf, torch.int64, 1) == 1
    assert copied(sf, torch.float32, 1) == 0           # roots of 4 MB: they nearly fit an L2
    assert copied(sf, torch.float32, 2) == 1 and copied(sf, torch.float64, 2) == 1
    assert copied(sf, torch.int32, 3) == 0             # three words a unit
    assert copied(sf, torch.float64, 4) == 0


def test_capture(graph):
    sf = S.StarForest(R, graph.iroot, None, graph.ranks).setup()
    assert copied(sf, torch.float64, 1) == 1
    root, leaf = torch.zeros(R, dtype=torch.float64, device="cuda"), torch.zeros(L, dtype=torch.float64, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sf.bcast(root, leaf)
        assert sf.choices()["last_bcast_copied"] == 0


def test_moves_between_streams(graph):
    """Two streams have a copy each; a third gets one once the calls of its
    last stream have completed."""
    sf = S.StarForest(R, graph.iroot, None, graph.ranks).setup()
    main, side, third = torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream()
    roots = [torch.randn(R, dtype=torch.float64, device="cuda") for _ in range(2)]
    index = torch.from_numpy(graph.iroot).cuda()
    leaf = torch.zeros(L, dtype=torch.float64, device="cuda")

    def call(stream, k):
        leaf.zero_()
        torch.cuda.synchronize()
        sf.bcast(roots[k], leaf, stream=stream)
        took = sf.choices()["last_bcast_copied"]
        torch.cuda.synchronize()
        assert torch.equal(leaf, roots[k][index])
        return took

    assert call(side, 0) == 1                          # a warm-up on a side stream
    for k in range(3):
        assert call(main, k & 1) == 1
    assert call(third, 1) == 1                         # the main stream's, whose calls have completed
    assert call(side, 0) == 1
    for _ in range(20):
        assert call(side, 1) == 1 and call(third, 0) == 1
    assert call(main, 1) == 0                          # no event behind the owners' last calls yet
    assert call(third, 0) == 1                         # this one hands its copy on
    assert call(main, 1) == 1 and call(side, 0) == 1


def test_set_up_allocates(graph):
    """No Bcast allocates: the copy is part of the plan's device memory."""
    sf = S.StarForest(R, graph.iroot, None, graph.ranks).setup()
    touched = sf.choices()["degree_ordered"]
    small = S.StarForest(3, [2, 0, 2]).setup()         # (the first launch loads the library's kernels)
    small.bcast(torch.zeros(3, device="cuda"), torch.zeros(3, device="cuda"))
    assert sf.info()["device_bytes"] >= 32 * touched + 4 * (touched + L)
    for dtype, bs in ((torch.float64, 1), (torch.float64, 2), (torch.float32, 4)):
        root = torch.zeros((R, bs), dtype=dtype, device="cuda")
        leaf = torch.zeros((L, bs), dtype=dtype, device="cuda")
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        sf.bcast(root, leaf)
        torch.cuda.synchronize()
        assert sf.choices()["last_bcast_copied"] == 1 and torch.cuda.mem_get_info()[0] == free
