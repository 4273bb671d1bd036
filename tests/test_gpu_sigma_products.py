"""The products of the order basis with few rows: the schoolbook tiles of four
coefficients a lane against the NTT, and the memory a basis takes."""
import numpy as np
import pytest

import synth
from test_gpu_transpose_lines import pool_bytes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

M31 = 2**31 - 1


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def series(dev, m, n, sigma, p):
    G = synth.vector(p + 3, m, m * n * sigma, 0, p - 1).reshape(m, n, sigma)
    return torch.from_numpy(G.astype(np.int32)).to(dev)


@pytest.mark.parametrize("p", [M31, 65521])
def test_four_coefficients_a_lane(dev, p):
    """Three rows, order 240,000 and no NTT: the last product has 235 tiles of 1,024 coefficients in each of nine
    entries, enough for the four-per-lane tiles; the basis is the NTT's."""
    from paper_1004_3719_amd import sigma_basis
    from paper_1004_3719_amd.ffx import set_ntt_threshold
    sigma = 240_000
    print("[case] four a lane", p, flush=True)
    G = series(dev, 3, 3, sigma, p)
    want, dw = sigma_basis(G, p, [0, 1, 2])
    set_ntt_threshold(0)
    try:
        got, dg = sigma_basis(G, p, [0, 1, 2])
    finally:
        set_ntt_threshold(1024)
    assert dw == dg and -(-(max(dg) - min(dg)) // 1024) < 3  # degrees close to one another: the last product is full
    assert max(dg) > 233 * 1024 and 9 * -(-(max(dg) + 1) // 1024) >= 2048
    assert torch.equal(want, got)


@pytest.mark.parametrize("m,n", [(1, 1), (2, 1), (3, 2)])
def test_few_rows_take_no_planes(dev, m, n):
    """Below four rows no product takes the matrix cores, and the workspace holds no operands for them."""
    from paper_1004_3719_amd import sigma_basis
    from paper_1004_3719_amd.ffx import set_ntt_threshold
    sigma = 8003
    G = series(dev, m, n, sigma, M31)
    set_ntt_threshold(0)
    try:
        used = pool_bytes(lambda: sigma_basis(G, M31, [0] * m))
    finally:
        set_ntt_threshold(1024)
    need = 2 * 4 * sigma * (m * m + m * n / 2)  # M1, R and M2 of a node and, half as long each time, of those below it
    print("[case] basis memory", m, n, used, need, flush=True)
    assert used <= need + 64 * 1024
