"""Captured MASTER solves in each form (one panel per work-group, one work-group, several for
many right-hand sides, chained and summed updates): every replay, with new inputs in the
captured buffers and eager solves in between, equals the eager result bitwise.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n_rhs", [(5, 300), (32, 1), (40, 65), (100, 3), (100, 40), (250, 2), (450, 1)])
def test_replays_equal_eager(m, n_rhs):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    g = torch.Generator().manual_seed(m)
    A, b = torch.randn(m, m, generator=g, dtype=torch.float64).cuda(), torch.randn(n_rhs, m, generator=g, dtype=torch.float64).cuda()
    x, work = torch.empty_like(b), torch.empty(m * (m + n_rhs), dtype=torch.float64, device="cuda")
    ctx = couple.couple_init(8)
    couple.couple_master_solve(ctx, A, b, work=work, out=x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        couple.couple_master_solve(ctx, A, b, work=work, out=x)
    for _ in range(4):
        A.copy_(torch.randn(m, m, generator=g, dtype=torch.float64))
        b.copy_(torch.randn(n_rhs, m, generator=g, dtype=torch.float64))
        want = couple.couple_master_solve(ctx, A, b)
        x.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(x, want)
