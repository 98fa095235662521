"""Float64 EB of several masks equals the one-mask calls bitwise where the one-mask form
changes: masks of one call on both sides of lmax 1000, and ranges of l3 with and without
a band, with the strips' product and with the tiles'.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _mask(torch, lmax, seed):
    rng = np.random.default_rng(seed)
    ell = np.arange(2 * lmax + 1.0)
    return [torch.as_tensor((ell + 1) ** -1.5 * np.exp(0.2 * rng.standard_normal(2 * lmax + 1))).cuda() for _ in range(3)]


@pytest.mark.parametrize("lmaxes", [[1003, 1002, 1001, 1000, 999, 998, 997], [999, 1000], [1000, 999, 999, 999, 999]])
def test_masks_on_both_sides_of_the_switch(lmaxes):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    masks = [_mask(torch, L, 10 * L + i) for i, L in enumerate(lmaxes)]
    ctx = couple.couple_init(max(lmaxes))
    for spectra in (("EB",), ("TT", "TE", "EE", "BB", "EB")):
        batch = couple.couple_matrix_batched(ctx, lmaxes, *[[m[x] for m in masks] for x in range(3)], spectra=spectra,
                                             precision="fp64")
        for L, m, K in zip(lmaxes, masks, batch):
            assert torch.equal(couple.couple_matrix(ctx, *m, L, spectra=spectra, precision="fp64"), K), (L, spectra)


@pytest.mark.parametrize("lmax,lo,hi", [(64, 0, 128), (1100, 0, 1099), (1100, 0, 1100), (1100, 1099, 1200), (1100, 1100, 1200),
                                        (2500, 0, 300), (2500, 100, 5000), (3000, 2400, 5000)])
def test_ranges_on_both_sides_of_the_switch(lmax, lo, hi):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    masks = [_mask(torch, lmax, lmax + i) for i in range(2)]
    ctx = couple.couple_init(lmax)
    batch = couple.couple_band_batched(ctx, lo, hi, *[[m[x] for m in masks] for x in range(3)], lmax, spectra=("EB",),
                                       precision="fp64")
    for i, m in enumerate(masks):
        assert torch.equal(couple.couple_band(ctx, lo, hi, *m, lmax, spectra=("EB",), precision="fp64"), batch[i]), i
