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
