"""The float64 whole-triangle kernels at the edges of their tiles and at each size
where the dispatch changes, against the multi-mask strips.

couple_matrix and couple_matrix_batched (and the band forms) promise the same
bits in float64, and reach them by different kernels: a tile's matrix product
and a diagonal strip's walk.  Two masks of one lmax are enough to send the
batched call through the strips, at every size.  So the comparison is exact.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# 16, 32, 64, 128: tile edges; 1000 .. 2900: where tiles take over from strips and grow
SIZES = [0, 1, 2, 3, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 999, 1000, 1150, 1250, 1399, 1400, 1401, 2399, 2400, 2700,
         2899, 2901]
ALL = ("TT", "TE", "EE", "BB", "EB")


def _windows(torch, lmax, seed):
    rng = np.random.default_rng(seed)
    ell = np.arange(2 * lmax + 1.0)
    out = []
    for _ in range(2):
        out.append([torch.as_tensor((ell + 1) ** -1.5 * np.exp(0.2 * rng.standard_normal(2 * lmax + 1))).cuda()
                    for _ in range(3)])
    return out


@pytest.mark.parametrize("lmax", SIZES + [6000, 8003])
def test_tiles_equal_strips(lmax):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    masks = _windows(torch, lmax, lmax)
    ctx = couple.couple_init(lmax)
    modes = [("TT",), ("EE",), ("TT", "EE"), ("TT", "TE", "EE"), ("EB",)] if lmax < 6000 else [("TT", "EE")] if lmax < 8000 else [("EE",)]
    for spectra in modes:
        batch = couple.couple_matrix_batched(ctx, [lmax, lmax], *[[m[x] for m in masks] for x in range(3)],
                                             spectra=spectra, precision="fp64")
        for m, K in zip(masks, batch):
            assert torch.equal(couple.couple_matrix(ctx, *m, lmax, spectra=spectra, precision="fp64"), K), spectra
        del batch


@pytest.mark.parametrize("lmax,lo,hi", [(33, 5, 40), (129, 128, 129), (1100, 0, 1100), (1405, 700, 2000), (1405, 2809, 4000)])
def test_l3_range_with_every_diagonal(lmax, lo, hi):
    """l3 restricted to [lo, hi] with hi >= lmax: no diagonal is left out, so the tiles run."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    masks = _windows(torch, lmax, lmax + hi)
    ctx = couple.couple_init(lmax + 7)
    batch = couple.couple_band_batched(ctx, lo, hi, *[[m[x] for m in masks] for x in range(3)], lmax, spectra=ALL,
                                       precision="fp64")
    for i, m in enumerate(masks):
        assert torch.equal(couple.couple_band(ctx, lo, hi, *m, lmax, spectra=ALL, precision="fp64"), batch[i])
