"""Few leaves on a wide leaf space: set-up takes memory and time by the leaves,
not by the slots, and the results are those of any other order."""
import subprocess
import sys

import numpy as np
import pytest

import oracle
from paper_2102_13018_amd import sf as S

WIDE = """
import resource
from paper_2102_13018_amd import sf as S
slots = [(1 << 28) - 1, 3, 1 << 20, 70000]
sf = S.StarForest(9, [4, 0, 7, 2], slots)
used = int(next(l for l in open("/proc/self/status") if l.startswith("VmSize")).split()[1]) * 1024
resource.setrlimit(resource.RLIMIT_AS, (used + (512 << 20),) * 2)
sf.setup(analyze_only=True)
assert sf.choices()["slot_ordered"] == 1
"""


def test_set_up_memory():
    """Half a GiB is room for the plan of four leaves, not for 4 bytes a slot."""
    r = subprocess.run([sys.executable, "-c", WIDE], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("nseg", [1, 3])
def test_results(nseg):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(4)
    nroots, n, space = 500, 3000, 3_000_000            # a thousand slots a leaf
    iroot, il = rng.integers(0, nroots, n), rng.choice(space, n, replace=False)
    sf = S.StarForest(nroots, iroot, il, np.arange(n) * nseg // n).setup(reduce_mode="deterministic")
    assert sf.choices()["slot_ordered"] == nseg
    root, leaf = rng.standard_normal(nroots), rng.standard_normal(int(il.max()) + 1)
    tr, tl = torch.from_numpy(root).cuda(), torch.from_numpy(leaf).cuda()
    sf.reduce(tl, tr, "sum")
    assert np.array_equal(tr.cpu().numpy(), oracle.reduce(nroots, iroot, il, leaf, root, "sum"))
    tr = torch.from_numpy(root).cuda()
    sf.bcast(tr, tl)
    assert np.array_equal(tl.cpu().numpy(), oracle.bcast(nroots, iroot, il, root, leaf, "replace"))
