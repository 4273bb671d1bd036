"""Column-sorted groups of a matrix whose entries are all +-1: no stored values,
and the same products as with them, bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def matrix(nrows, ncols, m, p_pm1):
    A = synth.rows(synth.spec(nrows, ncols, 61, len_kind=synth.LEN_ZIPF, len_a=1, len_b=min(3000, ncols), len_alpha=1.6,
                              col_kind=synth.COL_UNIFORM, p_pm1=p_pm1, val_lo=2, val_hi=m - 2 if m > 4 else 3))
    A.m = m
    if m == 2:
        A.val[:] = 1
    return A


@pytest.mark.parametrize("m", [2, 3, 251, 32749, 65536])
@pytest.mark.parametrize("shape", [(40_000, 33_001), (16_385, 16_384), (300, 50_000), (70_000, 1), (30_000, 30_000)])
@pytest.mark.parametrize("split", [True, False])
def test_all_pm1(dev, m, shape, split):
    from paper_1004_3719_amd import Matrix
    print("[case] all +-1", m, shape, split, flush=True)
    A = matrix(*shape, m, 1.0)
    orc = oracle.get()
    reorders = (False, True) if shape[0] == shape[1] else (False,)
    for reorder in reorders:
        M = Matrix.from_synth(A, col_sorted=1, split_pm1=split, reorder=reorder)
        I = M.info()
        assert I["sg_groups"] > 0
        for dtype in (torch.int32, torch.int64):
            x, xt = (synth.vector(62, k, n, 0, m - 1) for k, n in enumerate((A.ncols, A.nrows)))
            x[:2], xt[:2] = m - 1, m - 1
            y0, t0 = (synth.vector(63, k, n, 0, m - 1) for k, n in enumerate((A.nrows, A.ncols)))
            d = lambda v: torch.from_numpy(v.copy()).to(dtype).to(dev)
            assert np.array_equal(M.spmv(d(x)).cpu().numpy(), orc.spmv(A, x))
            got = M.spmv(d(x), alpha=m - 1, beta=m // 2, y=d(y0)).cpu().numpy()
            assert np.array_equal(got, orc.spmv(A, x, m - 1, m // 2, y0))
            assert np.array_equal(M.spmv_t(d(xt)).cpu().numpy(), orc.spmv_t(A, xt))
            got = M.spmv_t(d(xt), alpha=m - 1, beta=m // 2, y=d(t0)).cpu().numpy()
            assert np.array_equal(got, orc.spmv_t(A, xt, m - 1, m // 2, t0))
            if shape[0] == shape[1]:
                z = x
                for _ in range(3):
                    z = orc.spmv(A, z)
                assert np.array_equal(M.power(3, d(x)).cpu().numpy(), z)
        M.close()


def test_values_only_where_needed(dev):
    """4 bytes per entry word, and 2 for the value as soon as one entry is not +-1 or values are asked for."""
    from paper_1004_3719_amd import Matrix
    A = matrix(100_000, 100_000, 32749, 1.0)
    size = {}
    for name, val, split in (("pm1", None, True), ("values asked for", None, False), ("one other entry", 2, True)):
        if val is not None:
            A.val[7] = val
        M = Matrix.from_synth(A, col_sorted=1, split_pm1=split)
        size[name] = M.info()["sg_stream_bytes"]
        M.close()
    print("[case] column-sorted bytes", A.nnz, size, flush=True)
    assert size["values asked for"] == size["one other entry"]
    assert 1.4 < size["one other entry"] / size["pm1"] < 1.6
