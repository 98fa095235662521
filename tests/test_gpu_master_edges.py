"""MASTER solves with exchanges in nearly every column (dense Gaussian matrices) on either
side of each size at which the elimination changes form: one work-group or several (192),
chained or summed updates (400), rows per thread (512), panel widths (1024, 2048, 4096) and
the back substitution's blocks.  The bound is the backward error of Gaussian elimination
with partial pivoting, 64 m eps.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rhs", [1, 9])
@pytest.mark.parametrize("m", [191, 192, 193, 224, 225, 399, 400, 401, 512, 513, 544, 1023, 1024, 1025, 2048, 2049, 4096, 4097])
def test_exchanges_at_every_edge(m, n_rhs):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    g = torch.Generator().manual_seed(17 * m + n_rhs)
    A = torch.randn(m, m, generator=g, dtype=torch.float64).cuda()
    b = torch.randn(n_rhs, m, generator=g, dtype=torch.float64).cuda()
    ctx = couple.couple_init(8)
    x = couple.couple_master_solve(ctx, A, b)
    res = (A @ x.T - b.T).abs().max().item()
    scale = (A.abs().sum(1).max() * x.abs().max() + b.abs().max()).item()
    assert res <= 64 * m * np.finfo(float).eps * scale, res / scale
