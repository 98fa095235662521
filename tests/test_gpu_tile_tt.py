"""The temperature-only tile kernel at each of its shapes and where they change (2 x 2 MFMA
tiles per wave from lmax 2700, 4 x 2 from 6000, with sizes off the tiles' edges), and the
polarised patches at 2900: bitwise against the multi-mask strips, and some rows against the
oracle.
"""
import numpy as np
import pytest

from _parity import TOL_FP64, assert_parity

pytestmark = pytest.mark.gpu


def _mask(lmax, seed):
    rng = np.random.default_rng(seed)
    return [(np.arange(2 * lmax + 1) + 1.0) ** -1.5 * np.exp(0.2 * rng.standard_normal(2 * lmax + 1)) for _ in range(3)]


@pytest.mark.parametrize("lmax,spectra", [(L, ("TT",)) for L in (2699, 2700, 2701, 2751, 5999, 6000, 6001, 6079, 6143, 6144)] +
                         [(2900, ("EE",)), (2900, ("TT", "EE")), (2900, ("TT", "TE", "EE")), (2900, ("EB",))])
def test_shapes_equal_strips(lmax, spectra):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    masks = [[torch.as_tensor(w).cuda() for w in _mask(lmax, lmax + i)] for i in range(2)]
    ctx = couple.couple_init(lmax)
    batch = couple.couple_matrix_batched(ctx, [lmax, lmax], *[[m[x] for m in masks] for x in range(3)], spectra=spectra,
                                         precision="fp64")
    for m, K in zip(masks, batch):
        assert torch.equal(couple.couple_matrix(ctx, *m, lmax, spectra=spectra, precision="fp64"), K)


@pytest.mark.parametrize("lmax", [2701, 6079])
def test_rows_equal_the_oracle(oracle_bulk, lmax):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    W = _mask(lmax, 7)
    rows = np.array([0, 1, 63, 64, 127, 128, lmax // 2, lmax - 64, lmax - 1, lmax])
    Kr, Ar = oracle_bulk.coupling_rows(lmax, W[0], rows=rows, spectra=("TT",))
    ctx = couple.couple_init(lmax)
    K = couple.couple_matrix(ctx, torch.as_tensor(W[0]).cuda(), None, None, lmax, spectra=("TT",), precision="fp64")
    assert_parity(K[0][torch.as_tensor(rows).cuda()].cpu().numpy(), Kr[0], Ar[0], TOL_FP64, "TT at lmax %d" % lmax)
