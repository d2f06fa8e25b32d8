"""Which kernels a plan chooses (host analysis only): slot order, root order,
degree-ordered roots and the shared launch of chunk levels, either side of
each rule."""
import numpy as np
import pytest

from paper_2102_13018_amd import inputs
from paper_2102_13018_amd import sf as S


def choices(nroots, iroot, ilocal=None, ranks=None, **opts):
    return S.StarForest(nroots, iroot, ilocal, ranks).setup(analyze_only=True, **opts).choices()


def test_before_setup():
    with pytest.raises(S.SfError):
        S.StarForest(4, [0, 1, 2]).choices()


def test_slot_order():
    rng = np.random.default_rng(1)
    n = 5000
    iroot, il = rng.integers(0, 900, n), rng.permutation(n + 50)[:n]
    assert choices(900, iroot, il)["slot_ordered"] == 1
    assert choices(900, iroot, il, np.arange(n) // 1700)["slot_ordered"] == 3
    assert choices(900, iroot, il, hot_path="on")["slot_ordered"] == 0
    assert choices(900, iroot)["slot_ordered"] == 0
    assert choices(900, iroot, np.sort(il))["slot_ordered"] == 0          # ascending already
    assert choices(n, np.arange(n), il)["slot_ordered"] == 0              # a pattern on the root side


def test_root_order():
    rng = np.random.default_rng(2)
    n = 3000
    iroot = rng.permutation(2 * n)[:n]
    assert choices(2 * n, iroot)["rooted"] == 1
    assert choices(2 * n, np.arange(n))["rooted"] == 0                    # contiguous roots
    iroot[0] = iroot[1]
    assert choices(2 * n, iroot)["rooted"] == 0                           # a repeated root


def test_degree_order():
    R, L = 1_000_003, 2_500_001
    g = inputs.spmv_ghost(seed=90, nroots=R, nleaves=L, zipf_s=1.2, nseg=17)
    touched = np.unique(g.iroot).size
    assert choices(R, g.iroot, None, g.ranks)["degree_ordered"] == touched
    small = g.iroot[: (1 << 21) - 1]
    assert choices(R, small)["degree_ordered"] == 0                       # too few leaves
    flat = np.random.default_rng(3).integers(0, R // 8, L)
    assert choices(R, flat)["degree_ordered"] == 0                        # even degrees


def test_level_launch():
    deg = [1, 32, 33, 256, 257, 65536, 65537, 70000]
    iroot = np.repeat(np.arange(len(deg)), deg)
    assert choices(len(deg), iroot)["level_roots"] == 4                   # more than one chunk of 256
    assert choices(1, np.zeros(256, np.int64))["level_roots"] == 0
