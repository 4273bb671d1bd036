"""Products with several vectors at the edges of the lanes' pieces of rows:
widths about a piece (four 32-bit components, two of 64 bits), leading
dimensions that leave the wide loads at an element's alignment, tiles of the
most rows and of the most entries, rows over many runs and over many tiles, and
values at the ends of their range; bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

M31 = 2**31 - 1
FORMATS = ["STREAM", "SELL", "SELL_SORTED", "BAND_STREAM", "BAND_SELL_SORTED"]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def check(dev, A, s, dtype, ldx_extra, ldy_extra, off, top=False, **opts):
    from paper_1004_3719_amd import Matrix
    M = Matrix.from_synth(A, **opts)
    X = np.full((A.ncols, s), A.m - 1, np.int64) if top else synth.vector(81, 1, A.ncols * s, 0, A.m - 1).reshape(
        A.ncols, s)
    Y0 = synth.vector(81, 2, A.nrows * s, 0, A.m - 1).reshape(A.nrows, s)

    def place(v, extra):  # rows of s + extra elements, the first `off` elements into the buffer
        n, ld = v.shape[0], s + extra
        flat = torch.full((n * ld + off + 4,), A.m - 1, dtype=dtype, device=dev)
        t = flat[off:off + n * ld].view(n, ld)[:, :s]
        t.copy_(torch.from_numpy(v).to(dtype).to(dev))
        return t, flat

    Xd, _ = place(X, ldx_extra)
    Yd, flat = place(Y0, ldy_extra)
    before = flat.clone()
    M.spmm(Xd, alpha=A.m - 2, beta=A.m // 3, Y=Yd)
    assert np.array_equal(Yd.cpu().numpy(), oracle.get().spmm(A, X, A.m - 2, A.m // 3, Y0))
    Yd.copy_(torch.from_numpy(Y0).to(dtype).to(dev))
    assert torch.equal(flat, before)  # nothing beside the s components was written
    M.spmm(Xd, Y=Yd)
    assert np.array_equal(Yd.cpu().numpy(), oracle.get().spmm(A, X))
    M.close()


def mixed(nrows, ncols, m, seed, lmax=3000, val=2**40):
    A = synth.rows(synth.spec(nrows, ncols, seed, len_kind=synth.LEN_ZIPF, len_a=1, len_b=min(lmax, ncols),
                              len_alpha=1.6, col_kind=synth.COL_UNIFORM, band_lo=-2, band_hi=2, p_pm1=0.5, val_lo=-val,
                              val_hi=val))
    A.m = m
    return A


@pytest.mark.parametrize("m,dtype", [(65521, torch.int32), (M31, torch.int32), (M31, torch.int64)])
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("s", [2, 3, 4, 5, 6, 7, 8, 9, 11, 12, 15, 16])
def test_pieces(dev, s, fmt, m, dtype):
    A = mixed(1500, 1501, m, 31 + s)
    check(dev, A, s, dtype, s % 3, (s + 1) % 4, s % 2 + 1, fixed_format=fmt, tile_entries=256 if s % 2 else 1024)


@pytest.mark.parametrize("acc", ["int64", "fp64", "fp32"])
@pytest.mark.parametrize("s,m,tile_entries", [(2, 2039, 4096), (4, 2039, 256), (16, 2039, 4096)])
def test_largest_tiles(dev, acc, s, m, tile_entries):
    # 256 short rows to a tile, then rows of several tiles each, every term the largest
    n = 1100
    lens = np.where(np.arange(n) < 900, 4, 0)
    lens[950], lens[1000], lens[1001] = 4097, 9000, 1
    rowptr = np.concatenate([[0], np.cumsum(lens)])
    rng = np.random.default_rng(5)
    col = rng.integers(0, 9500, rowptr[-1])
    A = synth.Csr(n, 9500, rowptr.astype(np.int64), col.astype(np.int32), np.full(rowptr[-1], m - 1, np.int64))
    A.m = m
    check(dev, A, s, torch.int32, 0, 0, 0, top=True, fixed_format="STREAM", tile_entries=tile_entries, acc=acc)


@pytest.mark.parametrize("w", [1, 2, 3, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("n,L", [(1, 1), (255, 2), (256, 3), (513, 7)])
@pytest.mark.parametrize("fmt", [None, "STREAM", "SELL_SORTED"])
def test_gf2_sequence_blocks(dev, w, n, L, fmt):
    """Packed sequences about the 256-row blocks of the projection, the first iterations (whose folds lag
    by two) and every split of the bits over the lanes, against the product of the bit matrices."""
    from paper_1004_3719_amd import Matrix
    A = synth.rows(synth.spec(n, n, 17 + n, len_kind=synth.LEN_ZIPF, len_a=1, len_b=min(40, n), len_alpha=1.6,
                              col_kind=synth.COL_UNIFORM, band_lo=-2, band_hi=2, p_pm1=0.5, val_lo=-9, val_hi=9))
    A.m = 2
    M = Matrix.from_synth(A, fixed_format=fmt)
    U = torch.from_numpy(synth.vector(5, 1, n * w, -2**31, 2**31 - 1).reshape(n, w).astype(np.int32)).to(dev)
    V = torch.from_numpy(synth.vector(5, 2, n * w, -2**31, 2**31 - 1).reshape(n, w).astype(np.int32)).to(dev)
    S = M.sequence_gf2(U, V, L).cpu().numpy().view(np.uint32).reshape(L, 32 * w, w)
    bits = lambda x: np.unpackbits(x.cpu().numpy().view(np.uint8).reshape(n, 4 * w), axis=1, bitorder="little").astype(np.int64)
    u, W = bits(U), bits(V)
    for i in range(L):
        want = np.packbits((u.T @ W & 1).astype(np.uint8), axis=1, bitorder="little").view(np.uint32)
        assert np.array_equal(S[i], want), i
        W = oracle.get().spmm(A, W)
    M.close()


@pytest.mark.parametrize("xcd", [0, 1])
@pytest.mark.parametrize("fmts", [("SELL", "STREAM"), ("SELL",), ("STREAM",)])
def test_batch_kinds_of_tiles(dev, fmts, xcd):
    """Batches of SELL tiles, of others and of both (each kind has its own kernels), fewer items than workgroups and
    queues without any: every width of the right-hand sides."""
    from paper_1004_3719_amd import Batch, Matrix
    As = [synth.c1(seed=40 + k, n=200 + 150 * k) for k in range(9)]
    mats = [Matrix.from_synth(A, fixed_format=fmts[k % len(fmts)]) for k, A in enumerate(As)]
    s = [1, 2, 3, 4, 5, 8, 9, 13, 16]
    B = Batch(mats, s, xcd=xcd, use_graph=False)
    xs = [synth.vector(6, k, A.ncols * s[k], 0, A.m - 1).reshape(A.ncols, s[k]) for k, A in enumerate(As)]
    for _ in range(2):
        ys = [torch.full((A.nrows, q), -5, dtype=torch.int32, device=dev) for A, q in zip(As, s)]
        B.spmm([torch.from_numpy(x.astype(np.int32)).to(dev) for x in xs], ys)
        for A, x, y in zip(As, xs, ys):
            assert np.array_equal(y.cpu().numpy(), oracle.get().spmm(A, x))
