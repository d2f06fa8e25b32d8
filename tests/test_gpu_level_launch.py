"""The chunk levels of a root at the largest size that shares a launch (8192
results of 256 leaves) and one leaf beyond it, and units of several elements."""
import numpy as np
import pytest

import oracle
from paper_2102_13018_amd import sf as S

MOST = 8192 * 256


@pytest.mark.parametrize("n,roots", [(MOST, 2), (MOST + 1, 0)])
def test_choice(n, roots):
    iroot = np.concatenate([np.zeros(n, np.int64), np.ones(300, np.int64), [2]])
    assert S.StarForest(3, iroot).setup(analyze_only=True).choices()["level_roots"] == roots


@pytest.mark.gpu
@pytest.mark.parametrize("n", [MOST, MOST + 1])
@pytest.mark.parametrize("partition", ["on", "off"])
@pytest.mark.parametrize("dtype,bs", [(np.float64, 1), (np.float32, 3), (np.float32, 7)])
def test_results(n, partition, dtype, bs):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(n % 7 + bs)
    iroot = np.concatenate([np.zeros(n, np.int64), np.full(70_000, 1), np.full(300, 2), [3]])
    shape = (lambda k: (k,) if bs == 1 else (k, bs))
    sf = S.StarForest(5, iroot).setup(reduce_mode="deterministic", partition=partition)
    root, leaf = (rng.standard_normal(shape(k)).astype(dtype) for k in (5, iroot.size))
    tl = torch.from_numpy(leaf).cuda()
    for op in ("sum", "min"):
        tr = torch.from_numpy(root).cuda()
        sf.reduce(tl, tr, op)
        assert np.array_equal(tr.cpu().numpy(), oracle.reduce(5, iroot, None, leaf, root, op)), op
