"""Products of matrices large and even enough for a wavefront per 64 rows: which
matrices take it, that its rounding error is no larger than that of lanes per
row, and infinities and NaN."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_2102_13018_amd import sf as S

pytestmark = pytest.mark.gpu
G = 64


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def matrix(rng, lens, ncols, band=0):
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(rowptr[-1])
    if band:
        at = np.repeat(np.arange(lens.size) * (ncols / lens.size), lens).astype(np.int64)
        cols = np.clip(at + rng.integers(-band, band + 1, n), 0, ncols - 1)
    else:
        cols = rng.integers(0, ncols, n)
    return rowptr, cols.astype(np.int32), rng.standard_normal(n)


def uneven(rng, nrows, short, long, part):
    return np.where(rng.random(nrows) < part, long, short)


# (rows, columns, entries a row as (least, most) or (short, long, share of long), band) -> (panels, sums)
@pytest.mark.parametrize("nrows,ncols,lens,band,want", [
    (G * 1536, 5000, (3, 9), 0, (1, 4)), (G * 1535, 5000, (3, 9), 0, (0, 0)),        # wavefronts
    (G * 1535 + 1, 5000, (9, 33), 0, (1, 8)), (G * 1600, 5000, (20, 65), 0, (0, 0)),  # the longest row
    (G * 1536, 5000, (4, 40, 0.1), 0, (0, 0)), (G * 4096, 5000, (4, 40, 0.1), 0, (1, 8)),
    (G * 4096, 5000, (11, 70, 0.1), 0, (1, 16)), (G * 4096, 5000, (11, 90, 0.02), 0, (0, 0)),
    (G * 2048, 5000, (25, 25), 0, (0, 0)), (G * 2048, 5000, (24, 24), 0, (1, 4)),     # the mean row
    (G * 4096, G * 4096, (1, 1), 0, (0, 0)),                                          # one entry a row
    (G * 2047, 700_000, (12, 16), 0, (0, 0)), (G * 2048, 700_000, (12, 16), 0, (2, 4)),  # panels
    (G * 2048, 1_300_000, (10, 30), 0, (4, 4)), (G * 2048, 3_000_000, (30, 34), 0, (8, 4)),
    (G * 2048, 1_300_000, (10, 30), 60, (1, 4)),                                      # a band
    (G * 2048, 700_000, (5, 5), 0, (0, 0)), (G * 2048, 700_000, (2, 9), 0, (1, 4))])  # one panel, a wide x
def test_choices_and_results(nrows, ncols, lens, band, want):
    rng = np.random.default_rng(nrows + ncols)
    ln = uneven(rng, nrows, *lens) if len(lens) == 3 else rng.integers(lens[0], lens[1] + 1, nrows)
    ln[0], ln[-1] = max(lens[:2]), max(lens[:2])
    M = matrix(rng, ln, ncols, band)
    A = S.Csr(nrows, ncols, *M)
    assert A.choices() == want
    x, y0 = rng.standard_normal(ncols), rng.standard_normal(nrows)
    tx = torch.from_numpy(x).cuda()
    scale = oracle.csr_spmv(M[0], M[1], np.abs(M[2]), np.abs(x)) + np.abs(y0)
    for acc in (False, True):
        ty = torch.from_numpy(y0).cuda()
        A.spmv(tx, ty, accumulate=acc)
        want_y = oracle.csr_spmv(*M, x, y0 if acc else None)
        # any order of n <= 90 products and sums: (n + 8 panels) roundings of at most 2^-53 of the scale,
        # on either side
        assert np.all(np.abs(ty.cpu().numpy() - want_y) <= 2 * 100 * 2.0 ** -53 * scale)


def test_row_too_long_for_a_panel():
    """Rows of 140 entries over four panels are taken, in one of them not."""
    rng = np.random.default_rng(8)
    nrows, ncols = G * 4096, 1_300_000
    ln = np.full(nrows, 30)
    ln[7] = 140
    M = matrix(rng, ln, ncols)
    assert S.Csr(nrows, ncols, *M).choices()[0] == 4
    M[1][M[0][7]:M[0][8]] = np.arange(140)
    A = S.Csr(nrows, ncols, *M)
    assert A.choices() == (0, 0)
    x, ty = rng.standard_normal(ncols), torch.zeros(nrows, dtype=torch.float64, device="cuda")
    A.spmv(torch.from_numpy(x).cuda(), ty)
    scale = oracle.csr_spmv(M[0], M[1], np.abs(M[2]), np.abs(x))
    assert np.all(np.abs(ty.cpu().numpy() - oracle.csr_spmv(*M, x)) <= 2 * 150 * 2.0 ** -53 * scale)


def lane_tree(rowptr, vals, xs, rows, lanes):
    """Sums of the given rows with that many lanes per row: a lane's products one
    after the other (fused), then halves added to halves."""
    L = np.longdouble
    out = np.zeros((rows.size, lanes))
    n = rowptr[rows + 1] - rowptr[rows]
    for k in range(int(n.max())):
        on = np.nonzero(k < n)[0]
        e = rowptr[rows[on]] + k
        out[on, k % lanes] = (L(vals[e]) * L(xs[e]) + L(out[on, k % lanes])).astype(np.float64)
    while lanes > 1:
        lanes //= 2
        out = out[:, :lanes] + out[:, lanes:2 * lanes]
    return out[:, 0]


# rows around each limit of the running sums, in one panel and in several
@pytest.mark.parametrize("nrows,ncols,short,long,part,lanes", [
    (G * 4096, 5000, 15, 32, 0.05, 16), (G * 4096, 5000, 15, 33, 0.05, 16), (G * 4096, 5000, 15, 64, 0.05, 32),
    (G * 4096, 5000, 15, 65, 0.05, 32), (G * 4096, 5000, 15, 90, 0.02, 32),
    (G * 4096, 5000, 23, 124, 0.005, 32), (G * 2048, 1_300_000, 15, 15, 0, 16), (G * 2048, 1_300_000, 15, 40, 0.05, 32),
    (G * 2048, 5000, 24, 24, 0, 32), (G * 2048, 5000, 5, 5, 0, 8)])
def test_error_no_larger_than_lanes_per_row(nrows, ncols, short, long, part, lanes):
    rng = np.random.default_rng(long + nrows)
    ln = uneven(rng, nrows, short, long, part)
    M = matrix(rng, ln, ncols)
    A = S.Csr(nrows, ncols, *M)
    assert A.choices()[0] > 0
    x = rng.standard_normal(ncols)
    y = torch.zeros(nrows, dtype=torch.float64, device="cuda")
    A.spmv(torch.from_numpy(x).cuda(), y)
    y = y.cpu().numpy()
    xs = x[M[1]]
    exact = np.add.reduceat(np.longdouble(M[2]) * np.longdouble(xs), M[0][:-1])
    mean = ln.mean()
    assert lanes // 2 < mean <= lanes
    rows = np.nonzero(ln == long)[0][:20000]
    assert rows.size > 1000
    err = lambda got: float(np.sqrt(((np.longdouble(got) - exact[rows]) ** 2).mean()))  # noqa: E731
    # the root mean square of 1000 rows scatters by 1 / sqrt(2000), on either side: three times that
    assert err(y[rows]) <= err(lane_tree(M[0], M[2], xs, rows, lanes)) * (1 + 3 * np.sqrt(1 / rows.size))


@pytest.mark.parametrize("long", [9, 40, 90])
def test_infinities_and_nan(long):
    rng = np.random.default_rng(long)
    nrows, ncols = G * 4096, 4000
    ln = uneven(rng, nrows, 15 if long > 64 else 4, long, 0.02)
    ln[:6], ln[1] = long, 1
    M = matrix(rng, ln, ncols)
    assert S.Csr(nrows, ncols, *M).choices()[0] == 1
    x = rng.standard_normal(ncols)
    special = M[0][:6]
    M[1][special] = np.arange(6)
    x[:6] = [np.inf, np.inf, np.nan, 0.0, 1e200, 2.0]
    M[2][special] = [2.0, -1.0, 1.0, np.inf, 1e200, np.inf]   # inf, -inf, NaN, inf * 0, overflow, inf
    x[6:] = rng.standard_normal(ncols - 6)
    M[1][M[1] < 6] = 7
    M[1][special] = np.arange(6)
    A = S.Csr(nrows, ncols, *M)
    for y0 in (np.zeros(nrows), np.where(np.arange(nrows) % 1000 == 999, np.inf, 1.0)):
        ty = torch.from_numpy(y0).cuda()
        A.spmv(torch.from_numpy(x).cuda(), ty, accumulate=True)
        with np.errstate(all="ignore"):
            want = oracle.csr_spmv(*M, x, y0)
        got = ty.cpu().numpy()
        assert np.array_equal(np.isnan(got), np.isnan(want))
        inf = np.isinf(want)
        assert np.array_equal(got[inf], want[inf]) and np.all(np.isfinite(got[np.isfinite(want)]))
