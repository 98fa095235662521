"""Equal rows on either side of the sizes at which the MASTER solve changes its update:
below 400 unknowns they cancel exactly, so the matrix is singular and everything NaN.
Each pair is tried early in the elimination and with one row in the last panel.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pair", ["first", "apart", "last"])
@pytest.mark.parametrize("m", [383, 384, 385, 390, 399])
def test_equal_rows_below_400_give_nan(m, pair):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    i, j = {"first": (0, 1), "apart": (7, m - 1), "last": (m - 2, m - 1)}[pair]
    g = torch.Generator().manual_seed(m + j)
    A = torch.randn(m, m, generator=g, dtype=torch.float64)
    A[j] = A[i]
    ctx = couple.couple_init(8)
    x = couple.couple_master_solve(ctx, A.cuda(), torch.ones(2, m, dtype=torch.float64).cuda())
    assert torch.isnan(x).all()
