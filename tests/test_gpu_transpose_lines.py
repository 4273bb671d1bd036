"""The lines between the two forms of the transposed product without a stored
A^T, from both sides, bit for bit against the oracle. The form a call takes is
seen from the memory it takes from the pool: a scatter's is 64-bit sums, and
the records of the other form are 8 bytes an entry and more."""
import ctypes

import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

M31 = 2**31 - 1
RESERVED, USED_HIGH = 5, 8  # hipMemPoolAttrReservedMemCurrent, hipMemPoolAttrUsedMemHigh


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def pool_bytes(f):
    """Bytes f() takes from the device's stream-ordered pool at its most."""
    hip = ctypes.CDLL("libamdhip64.so")
    pool, v = ctypes.c_void_p(), ctypes.c_uint64(0)
    torch.cuda.synchronize()
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), 0) == 0
    assert hip.hipMemPoolSetAttribute(pool, USED_HIGH, ctypes.byref(v)) == 0
    f()
    torch.cuda.synchronize()
    assert hip.hipMemPoolGetAttribute(pool, USED_HIGH, ctypes.byref(v)) == 0
    return v.value


def check(dev, A, s, binned, **opts):
    from paper_1004_3719_amd import Matrix
    M = Matrix.from_synth(A, **opts)
    X = synth.vector(51, s, A.nrows * s, 0, A.m - 1).reshape(A.nrows, s)
    Xd = torch.from_numpy(X).to(dev)
    Y = torch.empty((A.ncols, s), dtype=torch.int64, device=dev)
    used = pool_bytes(lambda: M.spmm_t(Xd, Y=Y))
    assert np.array_equal(Y.cpu().numpy(), oracle.get().spmm_t(A, X))
    sums = 8 * A.ncols * (1 << (s - 1).bit_length())
    nnz, n_band = M.info()["nnz"], M.info()["n_band"]
    M.close()
    print("[case] lines", A.nrows, A.ncols, nnz, s, "pool", used, "sums", sums, flush=True)
    if binned is not None:
        assert (used > sums + 4096 or used > 8 * nnz) if binned else used <= sums + 4096
    return nnz, n_band


def uniform(n, ncols, k, m=65521):
    A = synth.rows(synth.spec(n, ncols, 19, len_kind=synth.LEN_FIXED, len_a=k, col_kind=synth.COL_UNIFORM, p_pm1=0.4,
                              val_lo=1, val_hi=m - 1))
    A.m = m
    return A


def band(n, k, m=M31):
    A = synth.rows(synth.spec(n, n, 20, len_kind=synth.LEN_FIXED, len_a=0, col_kind=synth.COL_BANDED,
                              band_lo=-(k // 2), band_hi=k - 1 - k // 2, p_pm1=0.0, val_lo=1, val_hi=m - 1))
    A.m = m
    return A


@pytest.mark.parametrize("s,diagonals,binned", [(1, 5, False), (1, 40, False), (1, 64, False), (2, 31, False),
                                                (2, 40, True), (3, 10, False), (4, 12, True), (5, 5, True),
                                                (8, 9, True), (16, 4, True)])
def test_diagonals(dev, s, diagonals, binned):
    nnz, n_band = check(dev, band(30_001, diagonals), s, binned, fixed_format="BAND_SELL")
    assert nnz - n_band < nnz / 10


@pytest.mark.parametrize("s,ncols,binned", [(1, 300_000, True), (2, 200_000, True), (2, 600_000, False),
                                            (3, 60_000, True), (3, 300_000, False), (8, 20_000, True),
                                            (8, 100_000, False), (16, 30_000, True), (16, 150_000, False)])
def test_short_runs(dev, s, ncols, binned):
    """Rows of 300, each a batch of its own."""
    check(dev, uniform(2000, ncols, 300), s, binned)


@pytest.mark.parametrize("s,n,k,binned", [(1, 10_000, 12, False), (1, 10_000, 14, True), (1, 23_000, 11, False),
                                          (1, 24_000, 11, True),
                                          (2, 800, 10, None), (4, 900, 10, None), (5, 40, 10, None),
                                          (8, 60, 10, None), (9, 25, 10, None), (16, 30, 10, None)])
def test_small(dev, s, n, k, binned):
    """Both sides of the lines by transactions (the pool gives the smallest products' memory in one block)."""
    check(dev, uniform(n, n, k), s, binned)


@pytest.mark.parametrize("s", [3, 5, 9, 11, 15, 16])
def test_large_sums_are_packed(dev, s):
    """A scatter's temporary above 256 MiB holds s sums to an output row, not a power of two."""
    from paper_1004_3719_amd import Matrix
    ncols = (1 << 25) // (1 << (s - 1).bit_length()) + 1
    A = uniform(3000, ncols, 9, m=M31)
    A.col[:5] = [0, 1, ncols - 3, ncols - 2, ncols - 1]
    M = Matrix.from_synth(A)
    X = synth.vector(52, s, A.nrows * s, 0, A.m - 1).reshape(A.nrows, s)
    Xd = torch.from_numpy(X).to(dev)
    Y = torch.empty((ncols, s), dtype=torch.int64, device=dev)
    used = pool_bytes(lambda: M.spmm_t(Xd, Y=Y))
    print("[case] packed", s, ncols, used, flush=True)
    assert np.array_equal(Y.cpu().numpy(), oracle.get().spmm_t(A, X))
    M.close()
    assert used <= 8 * ncols * s + 4096


@pytest.mark.parametrize("s,opts", [(1, {"col_sorted": 0}), (1, {"col_sorted": 1}), (4, {"col_sorted": 0})])
def test_temporary_is_given_back(dev, s, opts):
    """The pool keeps a transposed product's temporary while the handle lives, and at most 64 MiB after it."""
    from paper_1004_3719_amd import Matrix
    hip = ctypes.CDLL("libamdhip64.so")
    pool, v = ctypes.c_void_p(), ctypes.c_uint64(0)
    torch.cuda.synchronize()
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), 0) == 0
    assert hip.hipMemPoolTrimTo(pool, ctypes.c_size_t(0)) == 0

    def reserved():
        assert hip.hipMemPoolGetAttribute(pool, RESERVED, ctypes.byref(v)) == 0
        return v.value

    before = reserved()
    A = uniform(400_000, 400_000, 25)
    M = Matrix.from_synth(A, **opts)
    X = torch.ones((A.nrows, s), dtype=torch.int32, device=dev)
    Y = M.spmm_t(X)
    torch.cuda.synchronize()
    held = reserved()
    Z = M.spmm_t(X)  # from what the pool kept
    torch.cuda.synchronize()
    assert torch.equal(Y, Z) and reserved() == held
    M.close()
    print("[case] pool", s, opts, before, held, reserved(), flush=True)
    assert reserved() <= max(before, 64 << 20)
    if not opts["col_sorted"]:
        assert held > 64 << 20
