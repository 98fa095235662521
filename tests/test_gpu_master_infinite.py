"""Right-hand sides with an infinity or values near the largest double: the solution's
infinities stay infinities with the sign of the quotient, and other right-hand sides keep
their finite solutions.

K is a positive diagonal, or that with a constant above it.  The elimination multiplies
row r of the right-hand side by zeros for the rows below, so an infinity stands in the last
row only (0 x inf is NaN), a large finite value, whose quotient overflows, in any row; the
rows below it, and the right-hand sides beside it, are checked bit for bit.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 2, 31, 64, 65, 150, 192, 500, 600])
@pytest.mark.parametrize("value", [np.inf, -np.inf, 1.5e308])
def test_infinite_quotients(m, value):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    rng = np.random.default_rng(m)
    diag = np.full(m, 0.5)
    b = rng.standard_normal((3, m))
    ctx = couple.couple_init(8)

    def solve(K, rhs):
        return couple.couple_master_solve(ctx, torch.as_tensor(K).cuda(), torch.as_tensor(rhs).cuda()).cpu().numpy()

    clean = solve(np.diag(diag), b)
    assert np.array_equal(clean, 2.0 * b)
    for r in sorted({0, m // 2, m - 1}) if np.isfinite(value) else [m - 1]:
        c = b.copy()
        c[1, r] = value
        x = solve(np.diag(diag), c)
        assert np.array_equal(x[[0, 2]], clean[[0, 2]]), r
        assert x[1, r] == np.copysign(np.inf, value), r
        assert np.array_equal(x[1, r + 1:], clean[1, r + 1:]), r
    if m > 1:
        y = solve(np.diag(diag) + 0.25 * np.triu(np.ones((m, m)), 1), c)
        assert y[1, m - 1] == np.copysign(np.inf, value) and y[1, m - 2] == -y[1, m - 1]
