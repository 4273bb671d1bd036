"""Matrices without columns: every entry point gives beta*y, and the empty x
(whose pointer is null) is not read. Also the transposes of matrices without
rows, whose stored form has no columns."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

M31 = 2**31 - 1
FORMATS = [None, "STREAM", "SELL", "SELL_SORTED", "BAND_STREAM", "BAND_SELL", "BAND_SELL_SORTED"]
ROWS = [1, 70, 5000]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def build(nrows, ncols, m, **opts):
    from paper_1004_3719_amd import Matrix
    A = synth.Csr(nrows, ncols, np.zeros(nrows + 1, np.int64), np.zeros(0, np.int32), np.zeros(0, np.int64), m=m)
    return Matrix.from_synth(A, **opts)


def check(dev, product, n, s, m, dtype):
    """product(X, Y, alpha, beta) on an empty X against beta*Y, for one vector (s None) or s."""
    shape = (n,) if s is None else (n, s)
    X = torch.empty((0,) + shape[1:], dtype=dtype, device=dev)
    assert X.data_ptr() == 0
    Y0 = synth.vector(5, 1, n * (s or 1), 0, m - 1).reshape(shape)
    for alpha, beta in ((1, 0), (m - 1, m // 2)):
        Y = torch.from_numpy(Y0).to(dtype).to(dev)
        product(X, Y, alpha, beta)
        assert np.array_equal(Y.cpu().numpy(), Y0 * beta % m)


@pytest.mark.parametrize("acc,m", [("auto", 2), ("auto", 65521), ("auto", 1_000_003), ("auto", M31), ("fp64", 65521),
                                   ("fp64c", 1_000_003), ("fp32", 2039), ("fp32c", 8191)])
@pytest.mark.parametrize("fmt", FORMATS)
def test_no_columns(dev, fmt, acc, m):
    print("[case] no columns", fmt, acc, m, flush=True)
    for n in ROWS:
        opts = dict(fixed_format=fmt, acc=acc, compact_x=1 if n == 70 else -1)
        A = build(n, 0, m, **opts)
        T = build(0, n, m, build_transpose=True, **opts)
        for dtype in (torch.int32, torch.int64):
            check(dev, lambda x, y, a, b: A.spmv(x, a, b, y), n, None, m, dtype)
            check(dev, lambda x, y, a, b: A.spmv_noalloc(x, a, b, y), n, None, m, dtype)
            check(dev, lambda x, y, a, b: T.spmv_t(x, a, b, y), n, None, m, dtype)
            for s in (1, 2, 3, 8, 16):
                check(dev, lambda x, y, a, b: A.spmm(x, a, b, y), n, s, m, dtype)
                check(dev, lambda x, y, a, b: T.spmm_t(x, a, b, y), n, s, m, dtype)
        assert len(A.block_times(torch.empty(0, dtype=torch.int32, device=dev))) == A.info()["nblocks"]
        A.close()
        T.close()


@pytest.mark.parametrize("m", [65521, M31])
def test_no_columns_other_forms(dev, m):
    """Without a stored transpose, and with column-sorted groups."""
    for n in ROWS:
        T = build(0, n, m)
        check(dev, lambda x, y, a, b: T.spmv_t(x, a, b, y), n, None, m, torch.int32)
        check(dev, lambda x, y, a, b: T.spmm_t(x, a, b, y), n, 5, m, torch.int64)
        if m <= 65536:
            A = build(n, 0, m, col_sorted=1)
            check(dev, lambda x, y, a, b: A.spmv(x, a, b, y), n, None, m, torch.int32)


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("w", [1, 2, 8, 16])
def test_no_columns_gf2(dev, fmt, w):
    for n in ROWS:
        A = build(n, 0, 2, fixed_format=fmt)
        Y = torch.full((n, w), -1, dtype=torch.int32, device=dev)
        A.spmm_gf2(torch.empty((0, w), dtype=torch.int32, device=dev), Y=Y)
        assert int(Y.abs().sum()) == 0


@pytest.mark.parametrize("x16", [0, 1])
@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("fmt", ["STREAM", "SELL"])
def test_no_columns_in_a_batch(dev, fmt, graph, x16):
    """Between matrices with columns, and last; chunks of one column among them."""
    import oracle
    from paper_1004_3719_amd import Batch, Matrix
    A = synth.c4_matrix(3, nmax=3000)
    widths, Ms = [1, 9, 4, 1], []
    for k in range(4):
        Ms.append(build(300, 0, A.m, fixed_format=fmt) if k % 2 else Matrix.from_synth(A, fixed_format=fmt))
    B = Batch(Ms, widths, use_graph=graph, compact_x=x16)
    X = [synth.vector(9, k, A.ncols * s, 0, A.m - 1).reshape(A.ncols, s) for k, s in enumerate(widths)]
    Xs = [torch.empty((0, s), dtype=torch.int32, device=dev) if k % 2 else
          torch.from_numpy(X[k].astype(np.int32)).to(dev) for k, s in enumerate(widths)]
    Ys = [torch.full((300 if k % 2 else A.nrows, s), -1, dtype=torch.int32, device=dev) for k, s in enumerate(widths)]
    for _ in range(2):
        B.spmm(Xs, Ys)
        for k in range(4):
            want = np.zeros((300, widths[k])) if k % 2 else oracle.get().spmm(A, X[k])
            assert np.array_equal(Ys[k].cpu().numpy(), want), k
            Ys[k].fill_(-1)
