"""Order bases of the orders that one launch handles, at the edges of its lanes
and of its elimination: the fewest and the most rows and columns, one order to
two launches' worth, residuals with no pivot, with a pivot in the last column
alone, with rows that are multiples of one another, shifts that leave the
order of the rows reversed or far apart, and the largest residues."""
import numpy as np
import pytest

import oracle.sigma as osig
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

M31 = 2**31 - 1


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def series(kind, m, n, sig, p):
    G = synth.vector(m * 100 + n * 10 + sig, 5, m * n * sig, 0, p - 1).reshape(m, n, sig)
    if kind == "top":
        G[:] = p - 1
    elif kind == "zero":
        G[:] = 0
    elif kind == "late":  # nothing but the last column, and only from the middle order on
        G[:, : n - 1] = 0
        G[:, :, : sig // 2] = 0
    elif kind == "multiples":
        for i in range(1, m):
            G[i] = G[0] * (i + 1) % p
    elif kind == "sparse":
        G[synth.vector(3, 9, m * n * sig, 0, 3).reshape(m, n, sig) > 0] = 0
    return G


@pytest.mark.parametrize("p", [2, 65521, M31, M31 - 18])
@pytest.mark.parametrize("kind", ["random", "top", "zero", "late", "multiples", "sparse"])
@pytest.mark.parametrize("m,n,sig,shift", [(1, 1, 1, "zero"), (3, 2, 5, "down"), (4, 4, 31, "zero"), (5, 1, 32, "up"),
                                           (15, 7, 17, "down"), (16, 8, 2, "far"), (16, 8, 31, "gen"),
                                           (16, 8, 32, "down"), (16, 1, 33, "far"), (16, 8, 63, "up")])
def test_leaf(dev, m, n, sig, shift, kind, p):
    from paper_1004_3719_amd import sigma_basis
    G = series(kind, m, n, sig, p)
    d0 = {"zero": [0] * m, "up": list(range(m)), "down": list(range(m, 0, -1)), "gen": [0] * (m // 2) + [1] * (m - m // 2),
          "far": [2**28 if i % 3 == 0 else i % 2 for i in range(m)]}[shift]
    M, d = sigma_basis(torch.from_numpy(G.astype(np.int32)).to(dev), p, d0)
    Mo, do = osig.mbasis(G, sig, d0, p)
    assert d == do
    assert np.array_equal(M.cpu().numpy().astype(np.int64), Mo)


@pytest.mark.parametrize("p", [65521, M31, M31 - 18])
@pytest.mark.parametrize("m,n,sig,kind", [(4, 1, 65, "top"), (4, 3, 130, "random"), (5, 5, 97, "top"), (7, 2, 200, "random"),
                                          (9, 8, 129, "sparse"), (13, 4, 260, "random"), (16, 8, 140, "top"),
                                          (16, 7, 518, "random"), (3, 3, 130, "random")])
def test_products(dev, m, n, sig, kind, p):
    """Products at the edges of the matrix-core form: the fewest rows it takes and one below, column
    counts about the powers of two, ragged lengths, residues at the ends of their range."""
    from paper_1004_3719_amd import sigma_basis
    G = series(kind, m, n, sig, p)
    d0 = [0] * (m - n) + [1] * n
    M, d = sigma_basis(torch.from_numpy(G.astype(np.int32)).to(dev), p, d0)
    Mo, do = osig.mbasis(G, sig, d0, p)
    assert d == do
    assert np.array_equal(M.cpu().numpy().astype(np.int64), Mo)


@pytest.mark.parametrize("p", [65521, M31])
def test_products_long(dev, p):
    """Convolutions of thousands of coefficients (several flushes of the byte sums, four coefficients to
    a wave) against the transforms: the same basis either way."""
    from paper_1004_3719_amd import ffx, sigma_basis
    G = torch.from_numpy(series("top", 16, 8, 20000, p).astype(np.int32))
    G[:, :, 1::2] = torch.from_numpy(series("random", 16, 8, 10000, p).astype(np.int32))
    G, d0 = G.to(dev), [0] * 8 + [1] * 8
    try:
        ffx.set_ntt_threshold(0)
        M, d = sigma_basis(G, p, d0)
        ffx.set_ntt_threshold(64)
        Mt, dt = sigma_basis(G, p, d0)
    finally:
        ffx.set_ntt_threshold(1024)
    assert d == dt and torch.equal(M, Mt)
