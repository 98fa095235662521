"""MASTER solves of few unknowns with one to many right-hand sides, on either side of each
size and count at which the form changes: one panel per work-group (up to 32 unknowns),
one work-group, several.

The bound is the backward error of Gaussian elimination with partial pivoting, 64 m eps
(dense Gaussian matrices, which exchange rows in nearly every column).  The solution may
overwrite the right-hand side, and equal rows give NaN, in every form.

Many right-hand sides cost no multiple of one: they are solved beside each other, so a
call with 2000 of them stays below five calls with one (20 to 40 in one work-group).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [(m, r) for m in (1, 2, 8, 9, 16, 17, 31, 32) for r in (1, 255, 256, 257)]
CASES += [(m, r) for m in (33, 48) for r in (8, 9, 16, 17, 63, 64, 65, 300)] + [(m, r) for m in (49, 64) for r in (16, 17, 33)]
CASES += [(m, r) for m in (65, 80) for r in (31, 32, 33)] + [(m, r) for m in (81, 128, 191) for r in (8, 9, 16, 17, 130)]


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.mark.parametrize("m,n_rhs", CASES)
def test_right_hand_sides(torch, m, n_rhs):
    from paper_2602_15605_amd import couple
    g = torch.Generator().manual_seed(1000 * m + n_rhs)
    A = torch.randn(m, m, generator=g, dtype=torch.float64).cuda()
    b = torch.randn(n_rhs, m, generator=g, dtype=torch.float64).cuda()
    ctx = couple.couple_init(8)
    x = couple.couple_master_solve(ctx, A, b)
    res = (A @ x.T - b.T).abs().max().item()
    scale = (A.abs().sum(1).max() * x.abs().max() + b.abs().max()).item()
    assert res <= 64 * m * np.finfo(float).eps * scale, res / scale
    over = b.clone()
    couple.couple_master_solve(ctx, A, over, out=over)
    assert torch.equal(over, x)
    assert torch.equal(couple.couple_master_solve_noalloc(ctx, A, b), x)
    if m > 1:
        A[m - 1] = A[m // 2 - 1]
        assert torch.isnan(couple.couple_master_solve(ctx, A, b)).all()


@pytest.mark.parametrize("n,n_rhs", [(1, 3), (4, 300), (16, 2), (17, 70), (40, 20), (40, 40), (95, 17)])
def test_polarised_block(torch, n, n_rhs):
    """[EE EB; EB BB], the same solve as of the matrix written out."""
    from paper_2602_15605_amd import couple
    g = torch.Generator().manual_seed(n)
    K = torch.randn(3, n, n, generator=g, dtype=torch.float64).cuda()
    b = torch.randn(n_rhs, 2 * n, generator=g, dtype=torch.float64).cuda()
    A = torch.cat([torch.cat([K[0], K[2]], 1), torch.cat([K[2], K[1]], 1)], 0).contiguous()
    ctx = couple.couple_init(8)
    assert torch.equal(couple.couple_master_solve(ctx, K, b, pol=True), couple.couple_master_solve(ctx, A, b))


@pytest.mark.parametrize("m", [4, 30, 100])
def test_many_take_no_multiple_of_one(torch, m):
    from paper_2602_15605_amd import couple
    g = torch.Generator().manual_seed(m)
    A = torch.randn(m, m, generator=g, dtype=torch.float64).cuda()
    ctx = couple.couple_init(8)
    best = []
    for r in (1, 2000):
        b = torch.randn(r, m, generator=g, dtype=torch.float64).cuda()
        x, work = torch.empty_like(b), torch.empty(m * (m + r), dtype=torch.float64, device="cuda")
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        times = []
        for _ in range(8):
            e0.record()
            for _ in range(10):
                couple.couple_master_solve(ctx, A, b, work=work, out=x)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        best.append(min(times))
    assert best[1] <= 5 * best[0], best
