"""The fill's tile edges: matrices at the sizes where the tile changes (16, 32 and 64 by the
entries that a launch writes, the large form from 5e7) and at the edges of a tile, against
the definition K[l1][l2] = (2 l2 + 1) Xi(l1, l2) with Xi symmetric, exact in float64.
"""
import pytest

pytestmark = pytest.mark.gpu

# one output switches at 774 and 2449, four at 387, 1224 and 3535
CASES = [(0, 1), (1, 4), (15, 1), (16, 1), (31, 4), (63, 1), (64, 4), (773, 1), (774, 1), (386, 4), (387, 4), (1223, 4),
         (1224, 4), (2448, 1), (2449, 1), (3534, 4), (3535, 4)]


@pytest.mark.parametrize("lmax,n_out", CASES)
def test_fill_is_the_scaled_symmetric_kernel(lmax, n_out):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    spectra = ("TT", "TE", "EE", "BB")[:n_out]
    w = 1.0 / (1.0 + torch.arange(2 * lmax + 1, dtype=torch.float64, device="cuda")) ** 2
    ctx = couple.couple_init(max(lmax, 1))
    K = couple.couple_matrix(ctx, w, w, w, lmax, spectra=spectra, precision="fp32c")
    X = couple.couple_matrix(ctx, w, w, w, lmax, spectra=spectra, precision="fp32c", xi=True)
    f = 2.0 * torch.arange(lmax + 1, dtype=torch.float64, device="cuda") + 1.0
    for k, x in zip(K, X):
        assert torch.equal(x, x.T)
        assert torch.equal(k, f * x)
    if lmax >= 2:
        assert (X[0] > 0).all()
