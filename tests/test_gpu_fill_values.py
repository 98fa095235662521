"""The fill's tiles against the oracle: whole rows of K at the sizes where the tile changes
(16, 32 and 64 by the entries that a launch writes, the large form from 4.2e7 entries of
one mask, 5e7 of several), among them the first and last rows of a tile, of an edge tile
and of the matrix.  A row crosses every tile column, so a wrong source, a swapped pair of
mirrored tiles or a wrong diagonal shows in it.  The bounds are float32 sums' (1e-6 of the
sum of the terms' magnitudes).
"""
import numpy as np
import pytest

from _parity import TOL_FP32C, assert_parity

pytestmark = pytest.mark.gpu

CASES = [(15, 1), (16, 1), (64, 4), (386, 4), (387, 4), (773, 1), (774, 1), (1223, 4), (1224, 4), (2448, 1), (2449, 1),
         (3239, 4), (3240, 4), (6479, 1), (6480, 1)]


def _rows(lmax):
    last = lmax // 64 * 64
    return np.unique([r for r in (0, 1, 15, 16, 31, 32, 63, 64, lmax // 2, last - 1, last, lmax - 1, lmax) if 0 <= r <= lmax])


def _window(lmax, seed):
    rng = np.random.default_rng(seed)
    return (np.arange(2 * lmax + 1) + 1.0) ** -1.5 * np.exp(0.2 * rng.standard_normal(2 * lmax + 1))


@pytest.mark.parametrize("lmax,n_out", CASES)
def test_rows_equal_the_oracle(oracle_bulk, lmax, n_out):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    spectra = ("TT", "TE", "EE", "BB")[:n_out]
    W = [_window(lmax, 3 * lmax + x) for x in range(3)]
    rows = _rows(lmax)
    Kr, Ar = oracle_bulk.coupling_rows(lmax, *W, rows=rows, spectra=spectra)
    ctx = couple.couple_init(lmax)
    K = couple.couple_matrix(ctx, *[torch.as_tensor(w).cuda() for w in W], lmax, spectra=spectra, precision="fp32c")
    K = K[:, torch.as_tensor(rows.astype(np.int64)).cuda(), :].cpu().numpy()
    for i, x in enumerate(spectra):
        assert_parity(K[i], Kr[i], Ar[i], TOL_FP32C, "%s at lmax %d" % (x, lmax))


@pytest.mark.parametrize("lmaxes", [[3000, 2000, 1999, 64, 63, 0], [2500, 2500, 1800]])
def test_masks_in_one_launch(oracle_bulk, lmaxes):
    """Masks of one call share a launch: 5.1e7 entries (the large form) and 4.7e7."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    spectra = ("TT", "EE", "BB")
    Ws = [[_window(L, 10 * i + x) for x in range(3)] for i, L in enumerate(lmaxes)]
    ctx = couple.couple_init(max(lmaxes))
    lists = [[torch.as_tensor(w[x]).cuda() for w in Ws] for x in range(3)]
    outs = couple.couple_matrix_batched(ctx, lmaxes, *lists, spectra=spectra, precision="fp32c")
    for L, W, K in zip(lmaxes, Ws, outs):
        rows = _rows(L)
        Kr, Ar = oracle_bulk.coupling_rows(L, *W, rows=rows, spectra=spectra)
        K = K[:, torch.as_tensor(rows.astype(np.int64)).cuda(), :].cpu().numpy()
        for i, x in enumerate(spectra):
            assert_parity(K[i], Kr[i], Ar[i], TOL_FP32C, "%s at lmax %d" % (x, L))
