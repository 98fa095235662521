"""Window values that are infinite, NaN or near the largest double in the float64
whole-triangle kernels: they reach exactly the elements whose sums hold that l3, l1 and
l2 with |l1 - l2| <= l3 <= l1 + l2 and the spectrum's parity of l1 + l2 + l3, at each tile
shape.  All other elements keep the bits of the call with 0 in that place.

A value of 1e300 gives TT 1e300 times the kernel of that l3 alone: one term beside others
below its last place, so the factors' roundings are the whole error (1e-12, the float64
bound elsewhere).  The polarised sums, formed before their scaling by c_l1 c_l2, overflow.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# one size per tile shape: TT with 1 x 1, 2 x 2 and 4 x 2 MFMA tiles, then 2 x 2, 4 x 2 and 4 x 4 patches
CASES = [(40, ("TT",)), (333, ("TT",)), (2701, ("TT",)), (6001, ("TT",)), (1420, ("TT", "EE")), (1420, ("TT", "TE", "EE", "EB")),
         (2401, ("EE", "EB")), (2401, ("TT", "TE", "EE")), (2901, ("TT", "EE")), (2901, ("TT", "TE", "EE", "EB")), (2901, ("EE",))]


@pytest.mark.parametrize("lmax,spectra", CASES)
def test_wild_values_reach_their_own_elements(lmax, spectra):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    rng = np.random.default_rng(lmax)
    ell = np.arange(2 * lmax + 1.0)
    W = [(ell + 1) ** -1.5 * np.exp(0.2 * rng.standard_normal(2 * lmax + 1)) for _ in range(3)]
    ctx = couple.couple_init(lmax)

    def matrix(l3, value, others=True):
        w = [x.copy() if others else np.zeros_like(x) for x in W]
        for x in w:
            x[l3] = value
        return couple.couple_matrix(ctx, *[torch.as_tensor(x).cuda() for x in w], lmax, spectra=spectra, precision="fp64")

    l = torch.arange(lmax + 1, device="cuda")
    s, d = l[:, None] + l[None, :], (l[:, None] - l[None, :]).abs()
    for l3 in (0, lmax // 2 + 1, lmax, 3 * lmax // 2, 2 * lmax):
        zero = matrix(l3, 0.0)
        inside = (d <= l3) & (l3 <= s)
        even = inside & ((s + l3) % 2 == 0)
        own = [inside & ~even if x == "EB" else even for x in spectra]
        for value in (np.nan, np.inf, -np.inf):
            K = matrix(l3, value)
            for x, k, z, m in zip(spectra, K, zero, own):
                assert torch.equal(torch.isfinite(k), ~m), (x, l3, value)
                assert torch.equal(k[~m], z[~m]), (x, l3, value)
                if x == "TT" and np.isinf(value):
                    assert (k[m] == value).all(), (l3, value)
        one, huge = matrix(l3, 1.0, others=False), matrix(l3, 1e300)
        for x, k, z, o, m in zip(spectra, huge, zero, one, own):
            assert torch.equal(k[~m], z[~m]), (x, l3)
            if x == "TT":
                assert ((k[m] / 1e300 - o[m]).abs() <= 1e-12 * o[m].abs() + 1e-290).all(), l3
        del zero, K, one, huge
