"""Transposed products without a stored A^T at the edges of their two forms:
batches (one chunk, ragged tails, long rows, SELL groups, diagonals), panels
(one column over a power of two, the most panels, one column more) and the
widths of the vectors, bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

M31 = 2**31 - 1


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def tdev(a, dev, dtype=torch.int64):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dtype).to(dev)


def check(dev, A, s, dtype=torch.int64, axpby=True, **opts):
    from paper_1004_3719_amd import Matrix
    M = Matrix.from_synth(A, **opts)
    assert not M.info()["has_transpose"]
    X = synth.vector(91, 1, A.nrows * s, 0, A.m - 1).reshape(A.nrows, s)
    Y0 = synth.vector(91, 2, A.ncols * s, 0, A.m - 1).reshape(A.ncols, s)
    a, b = (A.m - 2, A.m // 3) if axpby else (1, 0)
    # a leading dimension above s on both sides
    Xd = torch.zeros((A.nrows, s + 3), dtype=dtype, device=dev)[:, :s]
    Yd = torch.zeros((A.ncols, s + 2), dtype=dtype, device=dev)[:, :s]
    Xd.copy_(tdev(X, dev, dtype))
    Yd.copy_(tdev(Y0, dev, dtype))
    for _ in range(2):  # the second call on the scratch the first one left
        Yd.copy_(tdev(Y0, dev, dtype))
        M.spmm_t(Xd, alpha=a, beta=b, Y=Yd)
        assert np.array_equal(Yd.cpu().numpy(), oracle.get().spmm_t(A, X, a, b, Y0))
    if s == 1:
        assert np.array_equal(M.spmv_t(tdev(X[:, 0], dev, dtype)).cpu().numpy(), oracle.get().spmv_t(A, X[:, 0]))
    M.close()


def powerlaw(nrows, ncols, m, seed=7):
    A = synth.rows(synth.spec(nrows, ncols, seed, len_kind=synth.LEN_ZIPF, len_a=1, len_b=min(5000, ncols),
                              len_alpha=1.6, col_kind=synth.COL_UNIFORM, band_lo=-2, band_hi=2, p_pm1=0.5,
                              val_lo=-(2**40), val_hi=2**40))
    A.m = m
    return A


@pytest.mark.parametrize("m", [2, 65521, 65536, 1_000_003, M31])
@pytest.mark.parametrize("s", [1, 2, 3, 4, 8, 11, 16])
@pytest.mark.parametrize("fmt", ["STREAM", "SELL_SORTED", "BAND_STREAM", "BAND_SELL"])
def test_binned_forms(dev, m, s, fmt):
    print("[case] binned", m, s, fmt, flush=True)
    check(dev, powerlaw(40_000, 33_001, m), s, fixed_format=fmt, dtype=torch.int32 if s % 2 else torch.int64)


@pytest.mark.parametrize("s,ncols", [(1, 64), (1, 65), (1, 8193), (1, 16384 * 256), (1, 16384 * 256 + 1),
                                     (3, 4096 * 256), (3, 4096 * 256 + 1), (16, 1024), (16, 1025)])
def test_panel_edges(dev, s, ncols):
    print("[case] panels", s, ncols, flush=True)
    A = synth.rows(synth.spec(60_000, ncols, 11, len_kind=synth.LEN_FIXED, len_a=12, col_kind=synth.COL_UNIFORM,
                              p_pm1=0.3, val_lo=1, val_hi=65520))
    A.m = 65521
    check(dev, A, s)


@pytest.mark.parametrize("s", [1, 8])
def test_extreme_terms_one_column(dev, s):
    """Every entry and x the residue m - 1, every row in one of two columns: the largest sums."""
    n = 600_000
    col = np.zeros(n, np.int32)
    col[::2] = 16_384
    for m in (65536, M31):
        A = synth.Csr(n, 16_385, np.arange(n + 1, dtype=np.int64), col, np.full(n, m - 1, np.int64), m=m)
        from paper_1004_3719_amd import Matrix
        M = Matrix.from_synth(A, split_pm1=False)
        X = np.full((n, s), m - 1, np.int64)
        got = M.spmm_t(tdev(X, dev)).cpu().numpy()
        assert np.array_equal(got, oracle.get().spmm_t(A, X))
        M.close()


def test_reordered_and_scattered(dev):
    """A reordered handle (x and y gathered into the stored order) and a product below the binned form's size."""
    A = powerlaw(40_000, 40_000, 32749)
    check(dev, A, 1, reorder=True)
    check(dev, A, 5, reorder=True)
    B = powerlaw(900, 700, M31)
    for s in (1, 2, 3, 8, 9):
        check(dev, B, s)


@pytest.mark.parametrize("m", [2, 3, 32749, 65521, 65536])
@pytest.mark.parametrize("shape", [(40_000, 33_001), (16_385, 16_384), (300, 50_000), (70_000, 1), (1, 40_000)])
def test_column_sorted_groups(dev, m, shape):
    """One vector on a handle with column-sorted groups: panels of 16,384 columns, chunks across their edges, fewer
    rows than groups, one column holding everything (whose 32-bit sums the index must refuse when they could wrap)."""
    print("[case] column sorted", m, shape, flush=True)
    A = powerlaw(*shape, m=m)
    check(dev, A, 1, col_sorted=1)
    check(dev, A, 1, dtype=torch.int32, col_sorted=1, split_pm1=False, axpby=False)


@pytest.mark.parametrize("m", [32749, 65536])
def test_column_sorted_largest_sums(dev, m):
    """Every entry and x the residue m - 1, in columns at and just above the length the 32-bit sums hold."""
    from paper_1004_3719_amd import Matrix
    longest = (2**32 - 1) // (3 * m)
    for n in (longest, longest + 1):
        A = synth.Csr(n, 2, np.arange(n + 1, dtype=np.int64), np.zeros(n, np.int32), np.full(n, m - 1, np.int64), m=m)
        M = Matrix.from_synth(A, col_sorted=1, split_pm1=False)
        x = np.full(n, m - 1, np.int64)
        assert np.array_equal(M.spmv_t(tdev(x, dev)).cpu().numpy(), oracle.get().spmv_t(A, x)), n
        M.close()


def test_column_sorted_reordered(dev):
    check(dev, powerlaw(40_000, 40_000, 32749), 1, col_sorted=1, reorder=True)


@pytest.mark.parametrize("m", [2, 65521, M31])
@pytest.mark.parametrize("s", [1, 2, 5, 8, 9, 16])
@pytest.mark.parametrize("fmt", ["STREAM", "SELL_SORTED", "BAND_STREAM", "BAND_SELL"])
def test_scattered_small(dev, m, s, fmt):
    """Below the fewest transactions that are binned: the atomics of one entry side by side."""
    A = powerlaw(201, 190, m, seed=23)
    assert A.nnz * ((s + 7) // 8) < 1 << 13
    check(dev, A, s, fixed_format=fmt)


def test_scattered_band(dev):
    """Almost only diagonals, one vector, more than 2^22 entries: atomics of adjacent lanes on adjacent sums."""
    n, w = 90_001, 48
    row = np.repeat(np.arange(n), w)
    col = (row + np.tile(np.arange(-20, w - 20), n)) % n
    rng = np.random.default_rng(3)
    rowptr = np.arange(0, n * w + 1, w, dtype=np.int64)
    A = synth.Csr(n, n, rowptr, col.astype(np.int32), rng.integers(2, M31 - 1, n * w))
    A.m = M31
    check(dev, A, 1, fixed_format="BAND_SELL")
