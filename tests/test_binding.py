"""The binding's argument checks on tensors: what is accepted and what is
refused does not depend on which of its two checks sees the buffer."""
import pytest

torch = pytest.importorskip("torch")

import numpy as np

from paper_2102_13018_amd import sf as S


class Dev:
    """A stand-in for a device tensor."""

    def __init__(self, n, dtype=torch.float64, cuda=True, contiguous=True):
        self.n, self.dtype, self.is_cuda, self.contiguous = n, dtype, cuda, contiguous

    def is_contiguous(self):
        return self.contiguous

    def numel(self):
        return self.n

    def element_size(self):
        return torch.empty(0, dtype=self.dtype).element_size()


@pytest.mark.parametrize("buf,ok", [
    (Dev(10), True), (Dev(11), True), (Dev(9), False), (Dev(10, cuda=False), False), (Dev(10, contiguous=False), False),
    (Dev(10, torch.float32), False), (Dev(20, torch.float32), False), (Dev(80, torch.uint8), True),
    (Dev(79, torch.int8), False), (Dev(10, torch.complex64), False), (1 << 20, True), (None, True), (object(), False)])
def test_buffers(buf, ok):
    sf = S.StarForest(10, np.arange(10))
    u = S.SfUnit(S.SF_F64, 1)
    for root, leaf in ((buf, Dev(10)), (Dev(10), buf)):
        if ok:
            sf._check(u, root, leaf)
        else:
            with pytest.raises(S.SfError) as e:
                sf._check(u, root, leaf)
            assert e.value.code == -1


def test_unit_of():
    for t, code in ((torch.float64, S.SF_F64), (torch.float32, S.SF_F32), (torch.int32, S.SF_I32),
                    (torch.int64, S.SF_I64), (torch.float16, S.SF_F16), (torch.bfloat16, S.SF_BF16)):
        for shape, bs in (((), 1), ((5,), 1), ((5, 3), 3), ((5, 2, 4), 8), ((0, 7), 7)):
            u = S.unit_of(torch.empty(shape, dtype=t))
            assert (u.dtype, u.bs) == (code, bs)
    for t in (torch.uint8, torch.complex64, torch.bool):
        with pytest.raises(KeyError):
            S.unit_of(torch.empty(3, dtype=t))
    a, b = S.unit_of(torch.empty(3)), S.unit_of(torch.empty(3))
    a.bs = 9
    assert b.bs == 1  # units are the caller's own
