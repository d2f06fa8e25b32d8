"""Set-up of permuted slots costs little more than set-up of the same leaves on
their own slots (host analysis only)."""
import time

import numpy as np
import pytest

from paper_2102_13018_amd import sf as S


def one(nroots, iroot, ilocal, ranks):
    sf = S.StarForest(nroots, iroot, ilocal, ranks)
    t0 = time.perf_counter()
    sf.setup(analyze_only=True)
    t = time.perf_counter() - t0
    sf.destroy()
    return t


@pytest.mark.parametrize("n,nseg", [(2500, 1), (16384, 1), (60000, 4)])
def test_permuted_slots(n, nseg):
    """Their order takes a walk over the slots and a count over some of the
    leaves; a sort per 64 leaves and one per segment took 3 to 10 times the plain
    set-up.  Fastest of 40 each, in turn."""
    rng = np.random.default_rng(1)
    iroot, il, ranks = rng.integers(0, n // 4, n), rng.permutation(n + n // 5)[:n], np.arange(n) * nseg // n
    plain, permuted = zip(*[(one(n // 4, iroot, None, ranks), one(n // 4, iroot, il, ranks)) for _ in range(40)])
    assert min(permuted) < 2.5 * min(plain)
