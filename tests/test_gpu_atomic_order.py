"""Atomic mode on permuted slots: the direct kernels walk the leaves in leaf
order where that has the roots together, in slot order elsewhere."""
import numpy as np
import pytest

import oracle
from paper_2102_13018_amd import sf as S

N = 30_011


def graph(kind, nseg=1):
    rng = np.random.default_rng(3)
    il = rng.permutation(N + 77)[:N]
    ranks = np.sort(rng.integers(0, nseg, N))
    if kind == "ascending":
        iroot = np.sort(rng.integers(0, N // 8, N))
    elif kind == "hot":      # a few roots with thousands of leaves, in ascending order
        iroot = np.sort((N // 8 * rng.random(N) ** 6).astype(np.int64))
    elif kind == "near":
        iroot = np.clip(np.arange(N) + rng.integers(-200, 200, N), 0, N - 1)
    else:
        iroot = rng.integers(0, N // 8, N)
    return int(iroot.max()) + 3, iroot, il, ranks


@pytest.mark.parametrize("kind,want", [("ascending", 1), ("hot", 1), ("near", 1), ("random", 0)])
def test_choice(kind, want):
    nroots, iroot, il, ranks = graph(kind)
    assert S.StarForest(nroots, iroot, il, ranks).setup(analyze_only=True).choices()["atomic_leaf_order"] == want
    assert S.StarForest(nroots, iroot, None, ranks).setup(analyze_only=True).choices()["atomic_leaf_order"] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("nseg", [1, 5])
@pytest.mark.parametrize("kind", ["ascending", "hot", "near", "random"])
@pytest.mark.parametrize("dtype,bs", [(np.int64, 1), (np.int32, 3), (np.int32, 5)])
def test_results(kind, nseg, dtype, bs):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from helpers import check_fetch_chain
    nroots, iroot, il, ranks = graph(kind, nseg)
    rng = np.random.default_rng(bs)
    shape = (lambda n: (n,) if bs == 1 else (n, bs))
    sf = S.StarForest(nroots, iroot, il, ranks).setup(reduce_mode="atomic", partition="off")
    space = int(il.max()) + 1
    root, leaf = rng.integers(-99, 99, shape(nroots)).astype(dtype), rng.integers(0, 99, shape(space)).astype(dtype)
    tl = torch.from_numpy(leaf).cuda()
    for op in ("sum", "max", "min"):
        tr = torch.from_numpy(root).cuda()
        sf.reduce(tl, tr, op)
        assert np.array_equal(tr.cpu().numpy(), oracle.reduce(nroots, iroot, il, leaf, root, op)), op
    tr, tu = torch.from_numpy(root).cuda(), torch.full(shape(space), -7, dtype=tl.dtype, device="cuda")
    sf.fetch_and_op(tr, tl, tu)
    got, upd = tr.cpu().numpy(), tu.cpu().numpy()
    hole = np.setdiff1d(np.arange(space), il)
    assert np.all(upd[hole] == -7)
    for c in range(bs):
        col = (lambda a: a if bs == 1 else a[:, c])
        check_fetch_chain(iroot, il, col(root), col(leaf), col(upd), col(got))
