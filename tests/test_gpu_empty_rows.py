"""STREAM tiles whose rows are mostly empty: several vectors bit for bit against
the oracle at the edges (entries in a tile's first and last rows, runs that
begin and end in long stretches of empty rows, empty tiles), and rows without
entries cost no more than rows with one."""
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


def matrix(lens, ncols, m, seed=3):
    rng = np.random.default_rng(seed)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    return synth.Csr(len(lens), ncols, rp, rng.integers(0, ncols, rp[-1]).astype(np.int32),
                     rng.integers(0, m, rp[-1]), m=m)


def lengths(kind, n):
    lens = np.zeros(n, np.int64)
    if kind == "ends":  # a tile's first and last rows only
        lens[::256], lens[255::256] = 3, 2
    elif kind == "gaps":  # 1 to 9 entries, then stretches of empty rows of every length
        at = np.cumsum(np.random.default_rng(1).integers(1, 400, n))
        at = at[at < n]
        lens[at] = np.arange(len(at)) % 9 + 1
    elif kind == "long":  # rows of several runs between empty ones
        lens[100::300] = 1500
    elif kind == "groups":  # tiles of as many entries as groups of lanes, one fewer and one more
        for k, ne in enumerate((63, 64, 65, 127, 128, 129, 255, 256, 257)):
            if 256 * k + 200 < n:
                lens[256 * k + 3], lens[256 * k + 200] = ne // 2, ne - ne // 2
    elif kind == "every":
        lens[::50] = 1
    return lens


@pytest.mark.parametrize("kind", ["ends", "gaps", "long", "groups", "every", "none"])
@pytest.mark.parametrize("m,acc", [(2, "auto"), (65521, "auto"), (M31, "auto"), (2039, "fp32"), (1_000_003, "fp64c")])
def test_mostly_empty_rows(dev, kind, m, acc):
    from paper_1004_3719_amd import Matrix
    print("[case] empty rows", kind, m, acc, flush=True)
    A = matrix(lengths(kind, 5000), 4999, m)
    M = Matrix.from_synth(A, fixed_format="STREAM", acc=acc)
    for s in (1, 2, 3, 4, 8, 11, 16):
        X = synth.vector(7, s, A.ncols * s, 0, m - 1).reshape(A.ncols, s)
        for dtype in (torch.int32, torch.int64):
            got = M.spmm(torch.from_numpy(X).to(dtype).to(dev))
            assert np.array_equal(got.cpu().numpy(), oracle.get().spmm(A, X)), (s, dtype)
    M.close()


@pytest.mark.parametrize("kind", ["ends", "gaps", "long", "groups", "every", "none"])
@pytest.mark.parametrize("n,diagonals", [(700, 0), (5000, 0), (700, 3), (5000, 3), (5000, 20)])
@pytest.mark.parametrize("m", [2, 65521, 1_000_003, M31])
def test_transposed_mostly_empty_rows(dev, kind, n, diagonals, m):
    """Without a stored transpose, below and above the line between atomics and records: entries that come after
    stretches of empty rows, alone and beside diagonals (a band from the first to the last column: entries outside)."""
    from paper_1004_3719_amd import Matrix
    print("[case] transposed empty rows", kind, n, diagonals, m, flush=True)
    A = matrix(lengths(kind, n), n, m)
    if diagonals:
        row, val = np.repeat(np.arange(n), diagonals), np.random.default_rng(4).integers(0, m, n * diagonals)
        col = row + np.tile(np.arange(diagonals) - 1, n)
        ok = (col >= 0) & (col < n)
        row = np.concatenate([np.repeat(np.arange(n), np.diff(A.rowptr)), row[ok]])
        col, val = np.concatenate([A.col, col[ok]]), np.concatenate([A.val, val[ok]])
        at = np.argsort(row, kind="stable")
        rp = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=n))]).astype(np.int64)
        A = synth.Csr(n, n, rp, col[at].astype(np.int32), val[at], m=m)
    for fmt in ("STREAM", "BAND_STREAM", "BAND_SELL"):
        M = Matrix.from_synth(A, fixed_format=fmt)
        for s in (1, 2, 3, 8, 16):
            X = synth.vector(8, s, n * s, 0, m - 1).reshape(n, s)
            got = M.spmm_t(torch.from_numpy(X).to(dev))
            assert np.array_equal(got.cpu().numpy(), oracle.get().spmm_t(A, X)), (fmt, s)
        M.close()


@pytest.mark.parametrize("s", [2, 4, 8])
def test_empty_rows_cost_no_more_than_full_ones(dev, s):
    """1,000,000 rows, one entry in fifty of them, take no longer than one in each (the same tiles)."""
    from paper_1004_3719_amd import Matrix
    n, us = 1_000_000, []
    X = torch.ones((n, s), dtype=torch.int32, device=dev)
    Y = torch.empty_like(X)
    for kind in ("every", "all"):
        lens = lengths(kind, n) if kind == "every" else np.ones(n, np.int64)
        M = Matrix.from_synth(matrix(lens, n, 65521), fixed_format="STREAM")
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        best = 1e9
        for _ in range(6):
            e0.record()
            for _ in range(20):
                M.spmm(X, Y=Y)
            e1.record()
            e1.synchronize()
            best = min(best, e0.elapsed_time(e1) * 50)
        us.append(best)
        M.close()
    print("[case] us per product: one row in fifty %.1f, every row %.1f" % tuple(us), flush=True)
    assert us[0] <= us[1]
