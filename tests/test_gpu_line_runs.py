"""Order-free operations of partitioned SFs where many windows' results meet in
one cache line of the roots (they take chunk levels) and where few do."""
import numpy as np
import pytest

import oracle
from paper_2102_13018_amd import sf as S

N = 1_300_000      # 159 windows of 8192 units, 318 of 4096


def graph(kind):
    rng = np.random.default_rng(6)
    if kind == "one":
        return 40, np.full(N, 17)
    if kind == "line":       # eight neighbours share a line of 8-byte and of 16-byte units
        return 40, rng.integers(16, 24, N)
    return 4000, rng.integers(0, 4000, N)


@pytest.mark.parametrize("kind", ["one", "line", "even"])
def test_runs(kind):
    nroots, iroot = graph(kind)
    small, wide = S.StarForest(nroots, iroot).setup(analyze_only=True, partition="on").choices()["line_runs"]
    windows = (N + 8191) // 8192, (N + 4095) // 4096
    if kind == "even":       # 325 leaves a root: two chunks of it at most, so two windows
        assert 0 < small <= 2 * 16 and 0 < wide <= 2 * 8
    else:                    # every window, twice where a root ends in it
        assert windows[0] <= small <= windows[0] + 8 and windows[1] <= wide <= windows[1] + 8


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["one", "line", "even"])
# atomics in the line: 159, 318, 636 and 954 without levels, 1272 and 1590 with them
@pytest.mark.parametrize("dtype,bs", [(np.float64, 1), (np.float64, 2), (np.int32, 2), (np.int32, 4), (np.float32, 4),
                                      (np.int64, 2)])
def test_results(kind, dtype, bs):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nroots, iroot = graph(kind)
    rng = np.random.default_rng(bs)
    shape = (lambda k: (k,) if bs == 1 else (k, bs))
    if np.dtype(dtype).kind == "i":
        root, leaf = (rng.integers(np.iinfo(dtype).min, np.iinfo(dtype).max, shape(k), dtype=dtype) for k in (nroots, N))
        ops = ("max", "min", "sum")
    else:
        root, leaf = (rng.standard_normal(shape(k)).astype(dtype) for k in (nroots, N))
        leaf.reshape(-1)[5::97] = -0.0
        ops = ("max", "min")
    for mode in ("deterministic", "auto"):
        sf = S.StarForest(nroots, iroot).setup(reduce_mode=mode, partition="on")
        tl = torch.from_numpy(leaf).cuda()
        for op in ops:
            tr = torch.from_numpy(root).cuda()
            sf.reduce(tl, tr, op)
            want = oracle.reduce(nroots, iroot, None, leaf, root, op)
            assert tr.cpu().numpy().tobytes() == want.tobytes(), op
